// grad.hip -- token-level OPD loss and its gradient with respect to the student logits.
//
// Eq. (2) (Sec. 3.1): L = - sum_t log pi_S(y_t) r_t 1_trainable(t), with
// r_t = log pi_T(y_t) - log pi_S(y_t) held constant (stop-gradient).  The
// trainable rows are the retained ones: units K0 .. stop of each rollout,
// including the unit that triggered the stop (Sec. 4.1, Algorithm 1).  For a
// retained row,  dL/ds_v = scale * r_t * (p_S(v) - [v = y_t]),  and the row's
// log-normaliser comes for free from the scoring pass: LSE_S = s_y - log pi_S(y),
// so p_S(v) = exp(s_v - s_y + log pi_S(y)).
//
// A row's wavefronts stream the student row once (16-byte non-temporal
// loads) and write the gradient row once; a row that is not retained is
// written as zeros without being read.  Columns ld - vocab of padding are not
// touched.  A small kernel first marks the retained rows.
#include "common.hpp"

namespace stride {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ uint32_t bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u) return (u >> 16) | ((u & 0xFFFFu) ? 0x40u : 0u);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// mask[i] = 1 if row i lies in a retained unit of its rollout, else 0.
__global__ __launch_bounds__(256) void grad_mask_kernel(stride_layout L, int32_t unit,
                                                        const int32_t *start, const int32_t *stop,
                                                        uint8_t *mask, uint32_t *flags) {
    const int64_t i = block_index<256>() * blockDim.x + threadIdx.x;
    if (i >= L.n_tokens) return;
    uint8_t m = 0;
    if (L.n_turns > 0 && L.turn_tok_off[0] <= i) {
        int64_t lo = 0, hi = L.n_turns;
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if (L.turn_tok_off[mid] <= i) lo = mid; else hi = mid;
        }
        const int64_t t = lo;
        if (i < L.turn_tok_off[t + 1] && L.n_rollouts > 0 && L.rollout_turn_off[0] <= t) {
            int64_t rlo = 0, rhi = L.n_rollouts;
            while (rhi - rlo > 1) {
                const int64_t mid = (rlo + rhi) >> 1;
                if (L.rollout_turn_off[mid] <= t) rlo = mid; else rhi = mid;
            }
            const int64_t t0 = L.rollout_turn_off[rlo], t1 = L.rollout_turn_off[rlo + 1];
            if (t < t1) {
                int64_t local, n;
                if (unit == STRIDE_UNIT_TURN) {
                    local = t - t0;
                    n = t1 - t0;
                } else {
                    local = i - L.turn_tok_off[t0];
                    n = L.turn_tok_off[t1] - L.turn_tok_off[t0];
                }
                int64_t k0 = start ? (int64_t)start[rlo] : 0;
                k0 = k0 < 0 ? 0 : (k0 > n ? n : k0);
                const int32_t s = stop ? stop[rlo] : -1;
                const int64_t last = (s >= 0 && (int64_t)s < n) ? (int64_t)s : n - 1;
                m = (local >= k0 && local <= last) ? 1 : 0;
            }
        } else {
            raise_flag(flags, STRIDE_FLAG_BAD_OFFSETS);
        }
    } else {
        raise_flag(flags, STRIDE_FLAG_BAD_OFFSETS);
    }
    mask[i] = m;
}

struct GradArgs {
    const void *student;
    const int32_t *ids;
    const float *logp_t;
    const float *logp_s;
    const uint8_t *mask;
    void *grad;
    float *loss;
    uint32_t *flags;
    int64_t n_rows;
    int64_t ld;
    int32_t vocab;
    float scale;
};

// W wavefronts per row, RW rows per workgroup: wavefront w handles the row's U-load chunks w, w + W, ...
// and every W-th word after the last whole chunk.  Every element's gradient depends only on that
// element, so nothing is merged and the bits do not depend on the split.  HBM bounds it (a read
// and a write stream); the row's first loads are issued before the sampled logit's two dependent
// ones are waited for.  launch_form has the choice of W and what it measured.
template <int DT, int W, int RW>
__global__ __launch_bounds__(W *RW *kWave) void opd_grad_kernel(GradArgs a) {
    static_assert(W == 1 || RW == 1, "a workgroup holds one row or one wavefront of each");
    constexpr int E = (DT == STRIDE_BF16) ? 8 : 4;
    constexpr int ES = (DT == STRIDE_BF16) ? 2 : 4;
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int sub = W == 1 ? 0 : wid;  // this wavefront's share of the row
    const int64_t row = block_index<W * RW * kWave>() * RW + (W == 1 ? wid : 0);
    if (row >= a.n_rows) return;
    const size_t off = (size_t)row * a.ld * ES;
    const u32x4 *src = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.student) + off);
    u32x4 *dst = reinterpret_cast<u32x4 *>(static_cast<char *>(a.grad) + off);
    const int64_t nvec = a.vocab / E;
    const int tail = a.vocab % E;
    const int32_t y = a.ids[row];
    const float lps = a.logp_s[row], lpt = a.logp_t[row];
    const bool retained = a.mask[row] != 0;
    const float r = lpt - lps;  // OPD reward, held constant
    const bool ok = (y >= 0) && (y < a.vocab) && (lps == lps) && (lpt == lpt) &&
                    (lps > -INFINITY) && (lpt > -INFINITY);
    if (sub == 0 && lane == 0) {
        if (a.loss) a.loss[row] = retained ? (ok ? -a.scale * lps * r : __builtin_nanf("")) : 0.0f;
        if (retained && !ok) raise_flag(a.flags, STRIDE_FLAG_NONFINITE);
    }
    if (!retained) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        for (int64_t k = (int64_t)sub * kWave + lane; k < nvec; k += (int64_t)W * kWave)
            __builtin_nontemporal_store(z, dst + k);
        if (tail && sub == 0 && lane == 0) {
            for (int j = 0; j < tail; ++j) {
                if (DT == STRIDE_BF16)
                    reinterpret_cast<uint16_t *>(dst + nvec)[j] = 0;
                else
                    reinterpret_cast<float *>(dst + nvec)[j] = 0.0f;
            }
        }
        return;
    }
    constexpr int U = 4;
    constexpr int64_t kStep = (int64_t)U * kWave;
    const int64_t nfull = nvec / kStep;  // whole U-load chunks
    u32x4 v[U];
    auto load = [&](int64_t c) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(src + c * kStep + u * kWave + lane);
    };
    if (sub < nfull) load(sub);
    __builtin_amdgcn_sched_barrier(0);
    // log-normaliser from the scoring pass: LSE_S = s_y - log pi_S(y)
    float sy = 0.0f;
    if (ok) {
        if (DT == STRIDE_BF16)
            sy = __uint_as_float((uint32_t)(reinterpret_cast<const uint16_t *>(src)[y]) << 16);
        else
            sy = reinterpret_cast<const float *>(src)[y];
    }
    const float c = ok ? a.scale * r : __builtin_nanf("");
    const float lse_l2 = (sy - lps) * kLog2e;
    const int64_t yv = ok ? (int64_t)(y / E) : -1;
    const int yj = ok ? y % E : 0;
    auto grad_vec = [&](const u32x4 v, int64_t vi) -> u32x4 {
        float x[E];
        if (DT == STRIDE_BF16) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[2 * i] = __uint_as_float(v[i] << 16);
                x[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(v[i]);
        }
        float g[E];
#pragma unroll
        for (int j = 0; j < E; ++j) g[j] = c * ex2(__builtin_fmaf(x[j], kLog2e, -lse_l2));
        if (vi == yv) {
#pragma unroll
            for (int j = 0; j < E; ++j)
                if (j == yj) g[j] -= c;
        }
        u32x4 o;
        if (DT == STRIDE_BF16) {
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = bf16_rne(g[2 * i]) | (bf16_rne(g[2 * i + 1]) << 16);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = __float_as_uint(g[i]);
        }
        return o;
    };
    for (int64_t c = sub; c < nfull; c += W) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t vi = c * kStep + u * kWave + lane;
            __builtin_nontemporal_store(grad_vec(v[u], vi), dst + vi);
        }
        if (c + W < nfull) load(c + W);
    }
    for (int64_t k = nfull * kStep + (int64_t)sub * kWave; k < nvec; k += (int64_t)W * kWave) {
        const int64_t vi = k + lane;
        if (vi < nvec) __builtin_nontemporal_store(grad_vec(__builtin_nontemporal_load(src + vi), vi), dst + vi);
    }
    if (tail && sub == 0 && lane == 0) {
        const u32x4 g = grad_vec(src[nvec], nvec);
        for (int j = 0; j < tail; ++j) {
            if (DT == STRIDE_BF16)
                reinterpret_cast<uint16_t *>(dst + nvec)[j] =
                    (uint16_t)(j & 1 ? (g[j >> 1] >> 16) : (g[j >> 1] & 0xFFFFu));
            else
                reinterpret_cast<float *>(dst + nvec)[j] = __uint_as_float(g[j]);
        }
    }
}

template <int DT, int W, int RW>
hipError_t launch_grad_form(const GradArgs &a, hipStream_t stream) {
    hipLaunchKernelGGL((opd_grad_kernel<DT, W, RW>), grid_of((a.n_rows + RW - 1) / RW, W * RW * kWave),
                       dim3(W * RW * kWave), 0, stream, a);
    return hipGetLastError();
}

// Wavefronts by the row's 16-byte words: as many as have words for their loads, so that fewer rows
// are read and written at a time; and short rows by their number, since few leave the chip idle.  Whole call (bits equal), eight wavefronts for every length ->
// the form taken here:
//   words 18,992 (bf16): 64 rows 26.6 -> 21.4 us, 2,000 rows 217 -> 199, 14,000 rows, two thirds of
//                        them retained, 1,394 -> 1,355, all retained 1,649 -> 1,610
//   words 25,000 (fp32), 3,000 rows: 448 -> 421 us; words 4,000, 20,000 rows: 391 -> 375
//   words 500, 20,000 rows: 70.8 -> 53.8 us; words 125, 30,000 rows: 64.1 -> 27.4
//   words 250: 256 rows 5.7 us either way (one 7.6), 1,024 rows 7.5 -> 7.0 (one 9.0), 4,096 rows 16.8 -> 12.3
//              (four 13.3); words 64: 256 rows 5.2 either way (one 5.4), 1,024 rows 6.1 -> 5.8 (one 5.6)
// Sixteen take 198 us against eight's 189 at 2,000 words, eight 105 against four's 95 at 1,000, but four
// 128 against eight's 120 at 1,030, where the words past four wavefronts' round of 1,024 are a round more.
template <int DT>
hipError_t launch_form(const GradArgs &a, hipStream_t stream) {
    const int words = a.vocab / (DT == STRIDE_BF16 ? 8 : 4);
    if (words < 256 && a.n_rows > (words < 64 ? 256 : 1024)) return launch_grad_form<DT, 1, 8>(a, stream);
    if (words <= 1024) return launch_grad_form<DT, 4, 1>(a, stream);
    if (words < 3072) return launch_grad_form<DT, 8, 1>(a, stream);
    return launch_grad_form<DT, 16, 1>(a, stream);
}

}  // namespace

hipError_t launch_opd_grad(const stride_layout &L, int32_t unit, int32_t dtype, int32_t vocab,
                           int64_t ld, const void *student, const int32_t *ids,
                           const float *logp_t, const float *logp_s, const int32_t *start,
                           const int32_t *stop, float scale, void *grad, float *loss,
                           uint32_t *flags, uint8_t *mask, hipStream_t stream) {
    if (L.n_tokens == 0) return hipSuccess;
    hipLaunchKernelGGL(grad_mask_kernel, grid_of((L.n_tokens + 255) / 256, 256), dim3(256), 0, stream, L, unit, start, stop,
                       mask, flags);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    GradArgs a;
    a.student = student;
    a.ids = ids;
    a.logp_t = logp_t;
    a.logp_s = logp_s;
    a.mask = mask;
    a.grad = grad;
    a.loss = loss;
    a.flags = flags;
    a.n_rows = L.n_tokens;
    a.ld = ld;
    a.vocab = vocab;
    a.scale = scale;
    if (dtype == STRIDE_BF16) return launch_form<STRIDE_BF16>(a, stream);
    return launch_form<STRIDE_F32>(a, stream);
}

}  // namespace stride
