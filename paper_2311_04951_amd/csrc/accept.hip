// Per-row softmax statistics and the modified rejection step of speculative sampling
// (Sections 3 and 4.3: the target accepts or rejects the draft's tokens so that the target
// distribution is recovered).
//
//   accept d_i  <=>  p_i(d_i) >= q_i(d_i)  or  fl32(u_i * q_i(d_i)) < p_i(d_i)      (prob. min(1, p/q))
//   on the first rejection: next ~ norm(max(0, p - q));  nothing rejected: next ~ p_{K+1}
//
// Sampling is an integer inverse CDF so that a parallel reduction and a sequential loop pick the same
// token: w_v = trunc(r_v * 2^32) (uint64), S = sum w_v, threshold = (u*2^24 * S) >> 24, token = the
// smallest v whose inclusive prefix exceeds the threshold.  Integer sums are associative, so the
// wavefront reductions below cannot change the answer.
//
// Row statistics (max, Z) use one pass over the vocabulary (online softmax) with wavefront shuffles;
// probabilities are defined by one fixed instruction sequence (prob_from_logit) so that the fused
// logits path and the materialised softmax produce identical bits.
#include "ss_device.h"
#include "ss_kernels.h"
#include <algorithm>
#include <type_traits>

namespace ss {

__device__ __forceinline__ float scaled_logit(float l, float inv_t) { return __fmul_rn(l, inv_t); }
// exp through the hardware's base-2 exponential (one rounded multiply, then v_exp_f32: about 2e-6 relative
// error at x = -30, far inside the tolerance on probabilities; the library routine costs five times the
// instructions and made these kernels ALU-bound)
__device__ __forceinline__ float fast_exp(float x) { return __builtin_amdgcn_exp2f(__fmul_rn(x, 1.4426950408889634f)); }
__device__ __forceinline__ float inv_norm(float Z) { return __fdiv_rn(1.0f, Z); }
// softmax probability of a logit given the row's (max, 1/Z): one fixed instruction sequence
__device__ __forceinline__ float prob_from_logit(float l, float inv_t, float mx, float invZ) {
    return __fmul_rn(fast_exp(__fsub_rn(scaled_logit(l, inv_t), mx)), invZ);
}

// ------------------------------------------------------------------ row statistics

__device__ __forceinline__ void online_merge(float &m, float &s, float m2, float s2) {
    const float mm = fmaxf(m, m2);
    s = s * fast_exp(m - mm) + s2 * fast_exp(m2 - mm);
    m = mm;
}

// one workgroup per row: stats[row] = (max_v x_v, sum_v exp(x_v - max)), x = logit * inv_t.
// Each thread keeps STATS_UNROLL independent 16-byte loads in flight per step (the row is streamed once
// and the kernel is bound by memory latency otherwise) and folds the step into its running (max, sum)
// with one rescale.
constexpr int STATS_UNROLL = 8;
// A row is cut into segments of STATS_SEG logits (a function of the vocabulary size alone, so every
// entry point computes a row's statistics with the same operations in the same order): one workgroup per
// segment, and the workgroup that finishes a row's last segment merges the segments in index order.
constexpr int STATS_SEG = 16384;
// (max_v x_v, sum_v exp(x_v - max)) of x[0 .. V) by a workgroup of 256 threads; valid in thread 0
__device__ __forceinline__ float2 segment_stats(const float *x, int V, float inv_t, bool vec) {
    float m = -INFINITY, s = 0.f;
    if (vec) {
        const f32x4 *x4 = reinterpret_cast<const f32x4 *>(x);
        const int n4 = V / 4;
        for (int i0 = threadIdx.x; i0 < n4; i0 += 256 * STATS_UNROLL) {
            f32x4 t[STATS_UNROLL];
#pragma unroll
            for (int j = 0; j < STATS_UNROLL; ++j) {
                const int i = i0 + 256 * j;
                t[j] = i < n4 ? __builtin_nontemporal_load(x4 + i) : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            }
            float mx = -INFINITY;
#pragma unroll
            for (int j = 0; j < STATS_UNROLL; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    t[j][e] = scaled_logit(t[j][e], inv_t);
                    mx = fmaxf(mx, t[j][e]);
                }
            if (mx == -INFINITY) continue;
            if (mx > m) {
                s *= fast_exp(m - mx);
                m = mx;
            }
            float add = 0.f;
#pragma unroll
            for (int j = 0; j < STATS_UNROLL; ++j) add += (fast_exp(t[j][0] - m) + fast_exp(t[j][1] - m)) + (fast_exp(t[j][2] - m) + fast_exp(t[j][3] - m));
            s += add;
        }
    } else {
        // rows without 16-byte alignment: the same with words, in whole lines, U of a thread's entries in flight (one load at a time, each
        // with an exponential behind a branch: 32 x K 10 x 50257 117.5 us a call of the logits entry, 50.6 now).  32 of them as long as there
        // are as many, then what the rest takes, and exponentials four at a time only where one of a wavefront's lanes has an entry: short rows
        // of a batch are bound by them (softmax of 1800 rows of 2051 | 4099, us, one load at a time 14.9 | 22.6, always 32 20.4 | 27.7, now
        // 14.3 | 21.5).  Ordinary loads: what writes the probabilities or draws the token reads the row again (the call of 32 x K 10 57.8 us with
        // non-temporal ones; only a softmax of more than the last-level cache holds gains by those, 1000 rows of 100001 259 us against
        // 272).  Which thread adds an entry depends on the row's length - and, where that is a multiple of 4, on the alignment of the
        // rows, which leads here or to the 16 bytes above.
        auto words = [&](int w0, auto u_, auto full_) { // entries w0 .. of a wavefront; FULL: all of the workgroup's 256 * U exist
            constexpr int U = decltype(u_)::value;
            constexpr bool FULL = decltype(full_)::value;
            const int lane = threadIdx.x & 63;
            float t[U], mx = -INFINITY;
#pragma unroll
            for (int j = 0; j < U; ++j) t[j] = x[FULL ? w0 + 256 * j + lane : min(w0 + 256 * j + lane, V - 1)];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                t[j] = FULL || w0 + 256 * j + lane < V ? scaled_logit(t[j], inv_t) : -INFINITY;
                mx = fmaxf(mx, t[j]);
            }
            if (mx == -INFINITY) { // nothing but masked entries - or a NaN (which a maximum passes over): the sum of a thread that has others becomes one
#pragma unroll
                for (int j = 0; j < U; ++j) s += t[j] != t[j] ? t[j] : 0.f;
                return;
            }
            if (mx > m) {
                s *= fast_exp(m - mx);
                m = mx;
            }
            float add = 0.f;
#pragma unroll
            for (int j = 0; j < U; j += 4)
                if (FULL || U <= 4 || w0 + 256 * j < V) {
                    float e[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int i = 0; i < (U < 4 ? U : 4); ++i) e[i] = fast_exp(t[j + i] - m);
                    add += (e[0] + e[1]) + (e[2] + e[3]);
                }
            s += add;
        };
        constexpr int MANY = 4 * STATS_UNROLL;
        const int own = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
        int v = 0;
        for (; v + 256 * MANY <= V; v += 256 * MANY) words(v + own, std::integral_constant<int, MANY>{}, std::true_type{});
        const int rest = V - v;
        if (rest > 256 * 16) words(v + own, std::integral_constant<int, MANY>{}, std::false_type{});
        else if (rest > 256 * 8) words(v + own, std::integral_constant<int, 16>{}, std::false_type{});
        else if (rest > 256 * 4) words(v + own, std::integral_constant<int, 8>{}, std::false_type{});
        else if (rest > 256 * 2) words(v + own, std::integral_constant<int, 4>{}, std::false_type{});
        else if (rest > 256) words(v + own, std::integral_constant<int, 2>{}, std::false_type{});
        else if (rest > 0) words(v + own, std::integral_constant<int, 1>{}, std::false_type{});
    }
    if (m == -INFINITY) s = 0.f; // a thread that saw nothing: exp(-inf - -inf) must not appear
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float m2 = __shfl_xor(m, o), s2 = __shfl_xor(s, o);
        if (m2 != -INFINITY) {
            if (m == -INFINITY) {
                m = m2;
                s = s2;
            } else {
                online_merge(m, s, m2, s2);
            }
        }
    }
    __shared__ float sm[4], ss_[4];
    if ((threadIdx.x & 63) == 0) {
        sm[threadIdx.x >> 6] = m;
        ss_[threadIdx.x >> 6] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float M = sm[0], S = ss_[0];
        for (int w = 1; w < 4; ++w)
            if (sm[w] != -INFINITY) {
                if (M == -INFINITY) {
                    M = sm[w];
                    S = ss_[w];
                } else {
                    online_merge(M, S, sm[w], ss_[w]);
                }
            }
        return make_float2(M, S);
    }
    return make_float2(0.f, 0.f);
}
// Statistics of segment `seg` of row x[0 .. V) and, by the workgroup that completes the row, of the row.
// cnt: the row's arrival counter (zero between launches); part: the row's nseg partial results.  Both are
// exchanged with agent-coherent accesses (the workgroups of a row run on different XCDs).
__device__ __forceinline__ void row_stats_segmented(const float *x, int V, float inv_t, int seg, int nseg, float2 *out, unsigned *cnt,
                                                    float2 *part) {
    const bool vec = (V % 4 == 0) && ((reinterpret_cast<uintptr_t>(x) & 15) == 0);
    const int lo = seg * STATS_SEG;
    const float2 r = segment_stats(x + lo, min(STATS_SEG, V - lo), inv_t, vec);
    if (threadIdx.x != 0) return;
    if (nseg == 1) {
        *out = r;
        return;
    }
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(part + seg), __builtin_bit_cast(unsigned long long, r), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt(0): the partial result is at the memory side before the arrival is counted
    if (__hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != (unsigned)(nseg - 1)) return;
    float M = -INFINITY, S = 0.f;
    for (int sgi = 0; sgi < nseg; ++sgi) {
        const float2 ps = __builtin_bit_cast(float2, ld_coh64(part + sgi));
        if (ps.x != -INFINITY) {
            if (M == -INFINITY) {
                M = ps.x;
                S = ps.y;
            } else {
                online_merge(M, S, ps.x, ps.y);
            }
        }
    }
    *out = make_float2(M, S);
    __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
int row_stats_segments(int V) { return std::max(1, (V + STATS_SEG - 1) / STATS_SEG); }
size_t row_stats_partial_bytes(int rows, int V) {
    const int nseg = row_stats_segments(V);
    return nseg == 1 ? 0 : sizeof(float2) * (size_t)rows * nseg;
}

// Two row sets in one launch (the target's and the draft's logits): rows [0, rows_a) are set a.  grid (segments, rows).
__global__ __launch_bounds__(256) void row_stats_kernel(const float *logits_a, int rows_a, float2 *stats_a, const float *logits_b,
                                                        float2 *stats_b, int V, float inv_t, unsigned *cnt, float2 *part) {
    const int id = blockIdx.y, nseg = gridDim.x;
    const bool first = id < rows_a;
    const int row = first ? id : id - rows_a;
    row_stats_segmented((first ? logits_a : logits_b) + (size_t)row * V, V, inv_t, blockIdx.x, nseg, (first ? stats_a : stats_b) + row,
                        cnt + id, part + (size_t)id * nseg);
}

// cnt: one arrival counter per row, zero before the launch (the kernel leaves them zero); part:
// row_stats_partial_bytes(rows, V) bytes.  Neither is touched when the vocabulary fits one segment.
void launch_row_stats(const float *logits, int rows, int V, float inv_t, float2 *stats, unsigned *cnt, float2 *part, hipStream_t st) {
    if (rows <= 0) return;
    hipLaunchKernelGGL(row_stats_kernel, dim3(row_stats_segments(V), rows), dim3(256), 0, st, logits, rows, stats, nullptr, nullptr, V, inv_t,
                       cnt, part);
}
void launch_row_stats2(const float *logits_a, int rows_a, float2 *stats_a, const float *logits_b, int rows_b, float2 *stats_b,
                       int V, float inv_t, unsigned *cnt, float2 *part, hipStream_t st) {
    if (rows_a + rows_b <= 0) return;
    hipLaunchKernelGGL(row_stats_kernel, dim3(row_stats_segments(V), rows_a + rows_b), dim3(256), 0, st, logits_a, rows_a, stats_a, logits_b,
                       stats_b, V, inv_t, cnt, part);
}

__global__ __launch_bounds__(256) void softmax_write_kernel(const float *logits, int V, float inv_t, const float2 *stats,
                                                            float *probs, int64_t ld) {
    const int row = blockIdx.y;
    const float2 st = stats[row];
    const float invZ = inv_norm(st.y);
    const size_t base = (size_t)row * V, obase = (size_t)row * ld;
    for (int v = blockIdx.x * 256 + threadIdx.x; v < V; v += gridDim.x * 256)
        probs[obase + v] = prob_from_logit(logits[base + v], inv_t, st.x, invZ);
}

void launch_softmax_write(const float *logits, int rows, int V, float inv_t, const float2 *stats, float *probs,
                          int64_t probs_ld, hipStream_t st) {
    if (rows <= 0) return;
    int gx = (V + 256 * 8 - 1) / (256 * 8);
    hipLaunchKernelGGL(softmax_write_kernel, dim3(gx, rows), dim3(256), 0, st, logits, V, inv_t, stats, probs, probs_ld);
}

// ------------------------------------------------------------------ a row of probabilities

struct RowSrc {
    const float *row;
    int from_logits;
    float inv_t, mx, invZ; // invZ = inv_norm(Z)
    __device__ __forceinline__ float conv(float x) const { return from_logits ? prob_from_logit(x, inv_t, mx, invZ) : x; }
    __device__ __forceinline__ float at(int v) const { return conv(row[v]); }
    // probabilities of v..v+3 (0 beyond V); v is a multiple of 4
    __device__ __forceinline__ void load4(int v, int V, bool vec, float (&out)[4]) const {
        if (vec && v + 3 < V) {
            const float4 t = *reinterpret_cast<const float4 *>(row + v);
            out[0] = conv(t.x);
            out[1] = conv(t.y);
            out[2] = conv(t.z);
            out[3] = conv(t.w);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = (v + e < V) ? conv(row[v + e]) : 0.f;
        }
    }
};

__device__ __forceinline__ unsigned long long fx_weight(float r) {
    return r > 0.f ? (unsigned long long)(r * 4294967296.0f) : 0ull;
}

template <bool RESID>
__device__ __forceinline__ void weights4(const RowSrc &P, const RowSrc &Q, int v, int V, bool vec,
                                         unsigned long long (&w)[4]) {
    float p[4];
    P.load4(v, V, vec, p);
    if (RESID) {
        float q[4];
        Q.load4(v, V, vec, q);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = fx_weight(fmaxf(__fsub_rn(p[e], q[e]), 0.f));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = fx_weight(p[e]);
    }
}

__device__ __forceinline__ unsigned long long shfl_xor_u64(unsigned long long x, int o) {
    const unsigned lo = __shfl_xor((unsigned)x, o), hi = __shfl_xor((unsigned)(x >> 32), o);
    return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long shfl_up_u64(unsigned long long x, int o) {
    const unsigned lo = __shfl_up((unsigned)x, o), hi = __shfl_up((unsigned)(x >> 32), o);
    return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long shfl_u64(unsigned long long x, int src) {
    const unsigned lo = __shfl((unsigned)x, src), hi = __shfl((unsigned)(x >> 32), src);
    return ((unsigned long long)hi << 32) | lo;
}

// threshold of the inverse CDF: floor(u * 2^24) * S >> 24 with a 128-bit product (u is a multiple of 2^-24)
__device__ __forceinline__ unsigned long long inv_cdf_threshold(float u, unsigned long long S) {
    const unsigned long long mant = (unsigned long long)(u * 16777216.0f);
    return (__umul64hi(mant, S) << 40) | ((mant * S) >> 24);
}

constexpr int SAMPLE_THREADS = 1024, SAMPLE_WAVES = SAMPLE_THREADS / 64;

// Integer inverse CDF over the range [r0, r1) of one row (r0 a multiple of 4) by a workgroup of NWAVES wavefronts.  Wave w owns a contiguous segment of the range; pass A sums every segment, pass B rescans
// the one segment that holds the threshold.  have_T: the threshold T (relative to the weight in front
// of r0, known to fall inside the range) is given; otherwise it is derived from u and the range's
// total, and -1 is returned when that total is 0.  Returns the token to every thread.
template <bool RESID, int NWAVES = SAMPLE_WAVES>
__device__ int block_inv_cdf(const RowSrc &P, const RowSrc &Q, int V, int r0, int r1, bool have_T, unsigned long long T,
                             float u, unsigned long long *sm_wave, int *sm_tok) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool vec = (V % 4 == 0) && ((reinterpret_cast<uintptr_t>(P.row) & 15) == 0) &&
                     (!RESID || (reinterpret_cast<uintptr_t>(Q.row) & 15) == 0);
    int seg = (r1 - r0 + NWAVES - 1) / NWAVES;
    seg = (seg + 255) & ~255;
    const int v_begin = min(r0 + wave * seg, r1), v_end = min(v_begin + seg, r1);

    // A range of up to four entries per lane and round stays in registers between the passes, all of it asked for at once (a round's loads
    // behind the one before, and again in pass B, were most of the finishing launch: logits entry of 64 x K 8 x 128256 104.7 -> 102.7 us,
    // 8 x 4 x 32000 22.1 -> 21.0).  As many rounds as the range has, and none for wavefronts behind its end (four for everyone, each with a
    // conversion to 64 bits: 1 x 8 x 5000 13.8 us one at a time, 15.0 with four, 13.4 now; probabilities 1 x 1 x 1000 6.8, 7.3, 7.0)
    constexpr int KEEP = 4;
    const bool keep = seg <= 256 * KEEP && r1 - r0 >= 4;
    unsigned long long sum = 0, kw[KEEP][4];
    if (keep) {
        const int own = v_begin + 4 * lane;
        auto fetch = [&](auto rounds_, auto vec_) { // (no branch between the loads: they are all in flight together)
            constexpr int ROUNDS = decltype(rounds_)::value;
            float kp[ROUNDS][4], kq[ROUNDS][4];
#pragma unroll
            for (int j = 0; j < ROUNDS; ++j) {
                if constexpr (decltype(vec_)::value) { // (r0 and r1 are multiples of 4)
                    const int v = min(own + 256 * j, r1 - 4);
                    const float4 a = *reinterpret_cast<const float4 *>(P.row + v), b = RESID ? *reinterpret_cast<const float4 *>(Q.row + v) : a;
                    kp[j][0] = a.x; kp[j][1] = a.y; kp[j][2] = a.z; kp[j][3] = a.w;
                    kq[j][0] = b.x; kq[j][1] = b.y; kq[j][2] = b.z; kq[j][3] = b.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int v = min(own + 256 * j + e, r1 - 1);
                        kp[j][e] = P.row[v];
                        kq[j][e] = RESID ? Q.row[v] : 0.f;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < KEEP; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    kw[j][e] = 0;
                    if (j < ROUNDS) {
                        const float w = RESID ? fmaxf(__fsub_rn(P.conv(kp[j][e]), Q.conv(kq[j][e])), 0.f) : P.conv(kp[j][e]);
                        kw[j][e] = own + 256 * j + e < v_end ? fx_weight(w) : 0ull;
                        sum += kw[j][e];
                    }
                }
        };
        auto fetch_rounds = [&](auto vec_) {
            if (seg <= 256) fetch(std::integral_constant<int, 1>{}, vec_);
            else if (seg <= 512) fetch(std::integral_constant<int, 2>{}, vec_);
            else fetch(std::integral_constant<int, KEEP>{}, vec_);
        };
        if (v_begin < v_end) { // (the same for the whole wavefront)
            if (vec) fetch_rounds(std::true_type{});
            else fetch_rounds(std::false_type{});
        }
    } else {
        for (int v = v_begin + 4 * lane; v < v_end; v += 256) {
            unsigned long long w[4];
            weights4<RESID>(P, Q, v, V, vec, w);
            sum += (w[0] + w[1]) + (w[2] + w[3]);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += shfl_xor_u64(sum, o);
    __syncthreads(); // protects sm_wave / sm_tok against a previous call in the same kernel
    if (lane == 0) sm_wave[wave] = sum;
    if (threadIdx.x == 0) *sm_tok = -1;
    __syncthreads();
    if (!have_T) {
        unsigned long long S = 0;
        for (int w = 0; w < NWAVES; ++w) S += sm_wave[w];
        if (S == 0) return -1;
        T = inv_cdf_threshold(u, S);
    }
    unsigned long long C = 0; // weight of the segments before mine
    for (int w = 0; w < wave; ++w) C += sm_wave[w];
    if (C <= T && T < C + sm_wave[wave]) { // wave-uniform: exactly one wave rescans its segment
        // true: the threshold is among these 256 entries
        auto find = [&](int v, const unsigned long long (&w)[4]) {
            const unsigned long long mine = (w[0] + w[1]) + (w[2] + w[3]);
            unsigned long long incl = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned long long t = shfl_up_u64(incl, o);
                if (lane >= o) incl += t;
            }
            const unsigned long long total = shfl_u64(incl, 63);
            if (C + total > T) {
                unsigned long long run = C + incl - mine;
                if (run <= T && T < run + mine) {
                    int tok = v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        run += w[e];
                        if (run > T) {
                            tok = v + e;
                            break;
                        }
                    }
                    *sm_tok = tok;
                }
                return true;
            }
            C += total;
            return false;
        };
        if (keep) {
            bool found = false;
#pragma unroll
            for (int j = 0; j < KEEP; ++j)
                if (!found) found = find(v_begin + 256 * j + 4 * lane, kw[j]);
        } else {
            for (int v0 = v_begin; v0 < v_end; v0 += 256) {
                const int v = v0 + 4 * lane;
                unsigned long long w[4] = {0, 0, 0, 0};
                if (v < v_end) weights4<RESID>(P, Q, v, V, vec, w);
                if (find(v, w)) break;
            }
        }
    }
    __syncthreads();
    return *sm_tok;
}

// (value, index) argmax of one row by the workgroup, lowest index on ties
__device__ int block_argmax(const RowSrc &P, int V, float *sm_val, int *sm_idx) {
    float best = -INFINITY;
    int bi = 0x7fffffff;
    for (int v = threadIdx.x; v < V; v += blockDim.x) {
        const float x = P.at(v);
        if (x > best || bi == 0x7fffffff) {
            best = x;
            bi = v;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float b2 = __shfl_xor(best, o);
        const int i2 = __shfl_xor(bi, o);
        if (b2 > best || (b2 == best && i2 < bi)) {
            best = b2;
            bi = i2;
        }
    }
    const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        sm_val[wave] = best;
        sm_idx[wave] = bi;
    }
    __syncthreads();
    best = sm_val[0];
    bi = sm_idx[0];
    for (int w = 1; w < nw; ++w)
        if (sm_val[w] > best || (sm_val[w] == best && sm_idx[w] < bi)) {
            best = sm_val[w];
            bi = sm_idx[w];
        }
    return bi;
}

// ------------------------------------------------------------------ the rejection step

__device__ __forceinline__ RowSrc make_row(const float *base, const float2 *stats, size_t row, int V, int from_logits,
                                           float inv_t) {
    RowSrc r;
    r.row = base + row * (size_t)V;
    r.from_logits = from_logits;
    r.inv_t = inv_t;
    r.mx = 0.f;
    r.invZ = 1.f;
    if (from_logits) {
        const float2 s = stats[row];
        r.mx = s.x;
        r.invZ = inv_norm(s.y);
    }
    return r;
}

// Leading accepted draft tokens of sequence b among its first `upto` positions, by the first `upto`
// threads of a workgroup (one gather of p_i(d_i), q_i(d_i) per thread, all in flight together); every
// thread gets the count.  Only the row statistics of positions up to the first rejection need to exist:
// whatever a later position computes from missing statistics cannot lower the minimum.
__device__ int block_accept_count(const AcceptArgs &a, int b, int upto, int *sm_rej) {
    if (threadIdx.x == 0) *sm_rej = upto;
    __syncthreads();
    if ((int)threadIdx.x < upto) {
        const int i = threadIdx.x;
        const int d = a.draft[b * a.K + i];
        bool acc = false;
        if (d < 0 || d >= a.V) { // cannot be validated on the host: flagged, treated as rejected
            atomicOr(a.status, 1);
        } else {
            const RowSrc P = make_row(a.p, a.p_stats, (size_t)b * (a.K + 1) + i, a.V, a.from_logits, a.inv_t);
            const RowSrc Q = make_row(a.q, a.q_stats, (size_t)b * a.K + i, a.V, a.from_logits, a.inv_t);
            const float pi = P.at(d), qi = Q.at(d);
            acc = (pi >= qi) || (__fmul_rn(a.u[b * (a.K + 1) + i], qi) < pi);
        }
        if (!acc) atomicMin(sm_rej, i);
    }
    __syncthreads();
    return *sm_rej;
}

// Row statistics in stages (logits entry).  Positions behind the first rejection of a sequence are never
// looked at by the method, so their rows need not be read: stage j covers positions [lo, hi) of every
// sequence (target rows lo .. hi-1, draft rows lo .. min(hi, K)-1) and, for lo > 0, a workgroup first counts
// the accepted tokens among positions < lo (their statistics exist if they are needed, see
// block_accept_count) and leaves when a rejection has already happened.  grid (rows of the stage, B).
__global__ __launch_bounds__(256) void row_stats_stage_kernel(AcceptArgs a, float2 *p_stats, float2 *q_stats, int lo, int hi, int nseg,
                                                              unsigned *cnt, float2 *part) {
    __shared__ int sm_rej;
    const int b = blockIdx.z, np = hi - lo;
    const bool target = (int)blockIdx.y < np;
    const int i = lo + (target ? blockIdx.y : blockIdx.y - np);
    if (lo > 0 && block_accept_count(a, b, lo, &sm_rej) < lo) return; // uniform over the workgroup
    const int row = target ? b * (a.K + 1) + i : b * a.K + i;
    const int id = target ? row : a.B * (a.K + 1) + row;
    row_stats_segmented((target ? a.p : a.q) + (size_t)row * a.V, a.V, a.inv_t, blockIdx.x, nseg, (target ? p_stats : q_stats) + row,
                        cnt + id, part + (size_t)id * nseg);
}

// stages of 2, 3, then all remaining positions (K + 1 target rows, K draft rows per sequence); cnt and part
// as for launch_row_stats with B * (2K + 1) rows
void launch_row_stats_staged(const AcceptArgs &a, float2 *p_stats, float2 *q_stats, unsigned *cnt, float2 *part, hipStream_t st) {
    if (a.B <= 0) return;
    const int nseg = row_stats_segments(a.V);
    int lo = 0;
    for (int stage = 0; lo <= a.K; ++stage) {
        int hi = std::min(lo + 2 + stage, a.K + 1);
        if (stage == 2 || a.K + 1 - hi < 2) hi = a.K + 1; // third stage, or a remainder not worth a launch
        const int np = hi - lo, nq = std::min(hi, a.K) - lo;
        hipLaunchKernelGGL(row_stats_stage_kernel, dim3(nseg, np + nq, a.B), dim3(256), 0, st, a, p_stats, q_stats, lo, hi, nseg, cnt, part);
        lo = hi;
    }
}

constexpr int PART_THREADS = 256, PART_UNROLL = 4;

// grid (nseg, B): the accepted count of sequence b, and the total weight of segment blockIdx.x of the
// row the next token is drawn from (residual at the first rejection, else the bonus row).  The
// vocabulary is cut into nseg segments so that a few sequences still fill the chip; integer partial
// sums make the split invisible in the result.  Bound by the two rows' bytes behind the chain draft -> probabilities -> row: a
// thread asks for the target's four 16-byte pieces of a round, then for the draft's four, none inside the bounds test of a piece (there,
// two were in flight; the logits call of 8 sequences x K 4 x 32000 25.5 -> 22.7 us, of 64 x K 8 x 128256 101.3 -> 99.4).  All eight
// asked for before the first is used measure the same.
__global__ __launch_bounds__(PART_THREADS) void accept_partial_kernel(AcceptArgs a, int seg_len, unsigned long long *partial) {
    __shared__ int sm_rej;
    __shared__ unsigned long long sm_part[PART_THREADS / 64];
    const int b = blockIdx.y, seg = blockIdx.x, nseg = gridDim.x;
    const int n = block_accept_count(a, b, a.K, &sm_rej);
    if (seg == 0 && threadIdx.x == 0) a.n_accepted[b] = n;
    const RowSrc P = make_row(a.p, a.p_stats, (size_t)b * (a.K + 1) + n, a.V, a.from_logits, a.inv_t);
    const bool resid = n < a.K;
    const RowSrc Q = resid ? make_row(a.q, a.q_stats, (size_t)b * a.K + n, a.V, a.from_logits, a.inv_t) : P;
    const bool vec = (a.V % 4 == 0) && ((reinterpret_cast<uintptr_t>(P.row) & 15) == 0) && ((reinterpret_cast<uintptr_t>(Q.row) & 15) == 0);
    const int r0 = min(seg * seg_len, a.V), r1 = min(r0 + seg_len, a.V);
    unsigned long long sum = 0;
    if (vec) { // (r0 and r1 are multiples of 4)
        for (int v0 = r0 + 4 * threadIdx.x; v0 < r1; v0 += 4 * PART_THREADS * PART_UNROLL) {
            float4 p4[PART_UNROLL], q4[PART_UNROLL];
#pragma unroll
            for (int j = 0; j < PART_UNROLL; ++j) p4[j] = *reinterpret_cast<const float4 *>(P.row + min(v0 + 4 * PART_THREADS * j, r1 - 4));
#pragma unroll
            for (int j = 0; j < PART_UNROLL; ++j) q4[j] = p4[j];
            if (resid) {
#pragma unroll
                for (int j = 0; j < PART_UNROLL; ++j) q4[j] = *reinterpret_cast<const float4 *>(Q.row + min(v0 + 4 * PART_THREADS * j, r1 - 4));
            }
#pragma unroll
            for (int j = 0; j < PART_UNROLL; ++j)
                if (v0 + 4 * PART_THREADS * j < r1) {
                    const float p[4] = {p4[j].x, p4[j].y, p4[j].z, p4[j].w}, q[4] = {q4[j].x, q4[j].y, q4[j].z, q4[j].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum += fx_weight(resid ? fmaxf(__fsub_rn(P.conv(p[e]), Q.conv(q[e])), 0.f) : P.conv(p[e]));
                }
        }
    } else {
        constexpr int U = 2 * PART_UNROLL; // (words, in whole lines)
        for (int v0 = r0 + threadIdx.x; v0 < r1; v0 += PART_THREADS * U) {
            float p[U], q[U];
#pragma unroll
            for (int j = 0; j < U; ++j) p[j] = P.row[min(v0 + PART_THREADS * j, r1 - 1)];
#pragma unroll
            for (int j = 0; j < U; ++j) q[j] = p[j];
            if (resid) {
#pragma unroll
                for (int j = 0; j < U; ++j) q[j] = Q.row[min(v0 + PART_THREADS * j, r1 - 1)];
            }
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (v0 + PART_THREADS * j < r1) sum += fx_weight(resid ? fmaxf(__fsub_rn(P.conv(p[j]), Q.conv(q[j])), 0.f) : P.conv(p[j]));
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += shfl_xor_u64(sum, o);
    if ((threadIdx.x & 63) == 0) sm_part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < PART_THREADS / 64; ++w) t += sm_part[w];
        partial[(size_t)b * nseg + seg] = t;
    }
}

// The segment that holds the threshold: the first of the nseg whose running sum passes it (bit i of `passed`).  None does where the
// threshold is not below the total (a uniform of 1 or more): the last one, in which nothing is found.
__host__ __device__ __forceinline__ int segment_of(unsigned long long passed, int nseg) { return passed ? __builtin_ctzll(passed) : nseg - 1; }
// For the tests (not part of the library's interface).
extern "C" int ss_dev_accept_segment(unsigned long long passed, int nseg) { return segment_of(passed, nseg); }

// one workgroup per sequence: locate the segment that holds the threshold and rescan it.  All residual
// weights zero (possible only through rounding): sample from p with the same uniform; all of those
// zero too: argmax.
__global__ __launch_bounds__(SAMPLE_THREADS) void accept_finish_kernel(AcceptArgs a, int seg_len, int nseg, const unsigned long long *partial) {
    __shared__ unsigned long long sm_wave[SAMPLE_WAVES];
    __shared__ int sm_tok;
    __shared__ float sm_val[SAMPLE_WAVES];
    __shared__ int sm_idx[SAMPLE_WAVES];
    const int b = blockIdx.x;
    const int n = a.n_accepted[b];
    const float u = a.u[b * (a.K + 1) + a.K];
    const RowSrc P = make_row(a.p, a.p_stats, (size_t)b * (a.K + 1) + n, a.V, a.from_logits, a.inv_t);
    const bool resid = n < a.K;
    const RowSrc Q = resid ? make_row(a.q, a.q_stats, (size_t)b * a.K + n, a.V, a.from_logits, a.inv_t) : P;
    // the segments' sums, one per lane (at most 16), and what is up to each of them
    const int lane = threadIdx.x & 63;
    const unsigned long long ps = lane < nseg ? partial[(size_t)b * nseg + lane] : 0ull;
    unsigned long long incl = ps;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        const unsigned long long x = shfl_up_u64(incl, o);
        if (lane >= o) incl += x;
    }
    const unsigned long long S = shfl_u64(incl, 15);
    int tok = -1;
    if (S != 0) {
        const unsigned long long T = inv_cdf_threshold(u, S); // (below S for a uniform in [0, 1))
        const int sgi = segment_of(__ballot(lane < nseg && T < incl), nseg); // the segment with C <= T < C + its sum
        const unsigned long long C = shfl_u64(incl - ps, sgi);
        const int r0 = min(sgi * seg_len, a.V), r1 = min(r0 + seg_len, a.V);
        tok = resid ? block_inv_cdf<true>(P, Q, a.V, r0, r1, true, T - C, u, sm_wave, &sm_tok)
                    : block_inv_cdf<false>(P, P, a.V, r0, r1, true, T - C, u, sm_wave, &sm_tok);
    } else if (resid) {
        tok = block_inv_cdf<false>(P, P, a.V, 0, a.V, false, 0, u, sm_wave, &sm_tok);
    }
    if (tok < 0) tok = block_argmax(P, a.V, sm_val, sm_idx);
    if (threadIdx.x == 0) a.next_token[b] = tok;
}

// segments per sequence: enough workgroups to fill the chip, of at least `least` vocabulary entries each
static int accept_segments(int B, int V, int least, int &seg_len) {
    int nseg = std::max(1, std::min(std::min(16, V / least), (1024 + B - 1) / std::max(B, 1)));
    seg_len = (V + nseg - 1) / nseg;
    seg_len = (seg_len + 1023) & ~1023; // multiple of the 4-wide loads of a whole workgroup
    nseg = (V + seg_len - 1) / seg_len;
    return std::max(nseg, 1);
}
constexpr int ACCEPT_SEG = 8192;

size_t accept_workspace_bytes(int B, int V) {
    int seg_len;
    return sizeof(unsigned long long) * (size_t)B * accept_segments(B, V, ACCEPT_SEG, seg_len);
}

// avail: bytes at `partial` (at least accept_workspace_bytes).  Where they hold more pairs than that minimum, segments go down to
// 2048 entries (two loads per thread; one sequence of 32000 entries: 9.2 -> 5.0 us with 11 segments instead of 3)
void launch_accept(const AcceptArgs &a, unsigned long long *partial, size_t avail, hipStream_t st) {
    if (a.B <= 0) return;
    int seg_len;
    int nseg = accept_segments(a.B, a.V, 2048, seg_len);
    if (sizeof(unsigned long long) * (size_t)a.B * nseg > avail) nseg = accept_segments(a.B, a.V, ACCEPT_SEG, seg_len);
    hipLaunchKernelGGL(accept_partial_kernel, dim3(nseg, a.B), dim3(PART_THREADS), 0, st, a, seg_len, partial);
    hipLaunchKernelGGL(accept_finish_kernel, dim3(a.B), dim3(SAMPLE_THREADS), 0, st, a, seg_len, nseg, partial);
}

// ------------------------------------------------------------------ top-p filter
//
// Top-p ("nucleus") and top-k selection of probability rows (Section 3 names both beside argmax; the arithmetic is fixed
// in the header of the C ABI): 32-bit integer weights, kept set = shortest prefix in (weight descending, index
// ascending) order whose weights reach the target (top-p) or the first k of that order (top-k), renormalised by one fp32
// division per element.  One workgroup per row looks for the weight of the last kept token:
//   1. a histogram over 2048 logarithmic bins (position of the leading bit, the six bits behind it), which spreads the weights of
//      a softmax over hundreds of bins (the top eleven bits of the weight put all but a few tokens into one);
//   2. the tokens of the bin that holds the boundary go to a list in LDS, usually some hundred, and the last kept one is found by
//      ranking them; where they are many, by digits of eleven of the remaining bits over that list - or over the row when they do not
//      fit (a row of equal weights);
//   3. one pass writes the row.
// All sums are integers, so the result does not depend on the order in which threads add.  A row of up to 32768 entries stays in
// LDS between the passes; a longer one is read again from the caches in each (16-byte loads where the rows allow).  Bound by the one compute unit that a row has; a split over several would need launches between the passes at
// 4 - 5 us each.  Measured at 5 rows of 32000 logits N(0, 2): top-k 35 -> 16 us (three digits over the row, five reads
// of it, before), top-p of what top-200 left 29 -> 9, of whole rows 18.
constexpr int TP_THREADS = 1024, TP_WAVES = TP_THREADS / 64, TP_BINS = 2048;

// Workgroup-wide exclusive prefix sum of one value per thread in thread order; also returns the total.
__device__ __forceinline__ unsigned long long block_excl_scan(unsigned long long mine, unsigned long long *sm_wave, unsigned long long &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long t = shfl_up_u64(incl, o);
        if (lane >= o) incl += t;
    }
    __syncthreads(); // sm_wave may still be read from a previous call
    if (lane == 63) sm_wave[wave] = incl;
    __syncthreads();
    unsigned long long before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < TP_WAVES; ++w) {
        const unsigned long long x = sm_wave[w];
        if (w < wave) before += x;
        total += x;
    }
    return before + incl - mine;
}

constexpr int TP_FITS = 32768; // longest row that stays in LDS
// entries of the boundary bin that fit LDS; up to which they are ranked one against all (200 take as long as the digits, 3.5 us)
constexpr int TP_LIST = 2048, TP_RANK = 192;
// Candidates: few enough tokens that hold every one that can be kept, found before the histogram, which then is theirs and not the row's
constexpr int TP_CAND = 1536;
// Most k for which the bound from the threads' largest tokens is looked for (more than that and the tokens above it are too many), and
// shortest row: of shorter ones a pass takes less than the bound (5 rows, top-k 40 | 200 | 512, us without and with it: 9001 entries 12.2 | 12.7 |
// 12.8 and 12.2 | 12.9 | 13.2, one aligned row of them 10.2 | 10.4 | 11.0 and 11.7 | 12.1 | 12.7; 64 rows of 16384 12.4 | 13.1 | 13.7 and 12.8 |
// 13.6 | 14.3, of 20000 14.2 | 15.2 | 23.6 and 13.3 | 14.2 | 19.6)
constexpr unsigned TP_FEW = 512;
constexpr int TP_FRONT_K = 18433;
// shortest row in which a top-p looks whether few tokens have a weight (its units are up to two per thread: nothing to save)
constexpr int TP_FRONT = 8193;
constexpr float TP_LEAST = 2.3283064365386963e-10f; // 2^-32, the smallest probability with a weight

// An entry's weight as the bits of a float, f = trunc(min(max(p * 2^32, 0), 2^32)): whole numbers of at most 24 significant bits, so
// f orders like the integer weight min(trunc(p * 2^32), 2^32 - 1) and is equal where that is (2^32 stands for 2^32 - 1).  Four
// instructions; a conversion to 64 bits takes some twenty, and a row has one compute unit to do them on.  The product is a
// fused multiply-add with +0, which makes +0 of a -0: a maximum of -0 and +0 may be either, and the bits of -0 would be the largest
// key of all (a comparison and a selection for that cost 3 - 9 % of the kernel, the multiply-add nothing).
__device__ __forceinline__ uint32_t tp_key(float p) { return f2u(truncf(fminf(fmaxf(__fmaf_rn(p, 4294967296.0f, 0.0f), 0.f), 4294967296.0f))); }
__device__ __forceinline__ uint32_t tp_weight(uint32_t key) { return key >= 0x4f800000u ? 0xffffffffu : (uint32_t)u2f(key); }
// monotone bin of a key >= 1.0: exponent and the six bits behind it.  2^0 .. 2^32 would be 2049 bins; 1.0 is alone in the 64 of its
// exponent, so everything above moves down by one
__device__ __forceinline__ int tp_bin(uint32_t key) { return max((int)(key >> 17) - 8129, 0); }
__device__ __forceinline__ uint32_t tp_bin_prefix(int bin) { return bin ? (uint32_t)bin + 8129u : 8128u; } // key >> 17 of the bin's keys
// x / Z rounded to nearest, for 2^-32 <= x < 1 and 2^-32 <= Z < 2^18, from rZ = 1 / Z rounded to nearest: two remainder steps, the
// first of which makes the quotient faithful and the second rounds it correctly (Markstein, "Computation of elementary functions
// on the IBM RISC System/6000 processor", 1990); nothing under- or overflows in that range.  Five instructions; the general
// division takes three times as many and changes the rounding mode twice, which made the writing pass the longest of the kernel.
__device__ __forceinline__ float tp_divide(float x, float Z, float rZ) {
    float q = __fmul_rn(x, rZ);
    q = __fmaf_rn(__fmaf_rn(-q, Z, x), rZ, q);
    return __fmaf_rn(__fmaf_rn(-q, Z, x), rZ, q);
}
// A row in units of four entries, unit i to thread i % TP_THREADS: neighbouring entries where 16-byte accesses are possible, else
// entries TP_THREADS apart (a wavefront's word loads then cover whole lines; four neighbouring words per lane took four times the
// requests: top-k of 5 rows of 50257 entries 49 -> 29 us).  Entry e of unit i:
template <bool VEC> __device__ __forceinline__ int tp_entry(int i, int e) { return VEC ? 4 * i + e : (i & ~(TP_THREADS - 1)) * 4 + e * TP_THREADS + (i & (TP_THREADS - 1)); }
template <bool VEC> __device__ __forceinline__ int tp_units(int V) { return VEC ? (V + 3) / 4 : (V + 4 * TP_THREADS - 1) / (4 * TP_THREADS) * TP_THREADS; }
template <bool VEC> __device__ __forceinline__ f32x4 tp_load4(const float *p, int i, int V) { // absent entries read as 0
    if (VEC && 4 * i + 3 < V) return *reinterpret_cast<const f32x4 *>(p + 4 * i);
    f32x4 q;
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = tp_entry<VEC>(i, e) < V ? p[tp_entry<VEC>(i, e)] : 0.f;
    return q;
}

// BY_COUNT = false: top-p, the histograms hold sums of weights and the selection looks for the weight at which the running
// sum reaches ceil(P24 * S / 2^24).  BY_COUNT = true: top-k (`P24` carries k, 1 <= k < V), the histograms hold counts and the
// selection looks for the weight of the k-th token (tokens without a weight are the tail of the order).
// FRONT: looks for candidates first.
template <bool BY_COUNT, bool VEC, bool FITS, bool FRONT>
__global__ __launch_bounds__(TP_THREADS) void top_p_filter_kernel(const float *probs, long long ld_in, int V, unsigned P24, float *out, long long ld_out) {
    typedef typename std::conditional<BY_COUNT, unsigned, unsigned long long>::type Bin;
    __shared__ Bin hist[TP_BINS];
    __shared__ unsigned long long sm_wave[TP_WAVES];
    __shared__ unsigned long long sm_above, sm_binw;
    __shared__ uint32_t list[TP_LIST];
    __shared__ int sm_bin, sm_cut, sm_n, sm_nc;
    __shared__ __align__(16) uint8_t sm_nz[TP_WAVES]; // (16 of them)
    __shared__ f32x4 row[FITS ? TP_FITS / 4 : TP_CAND / 4]; // (a longer row: the candidates' probabilities)
    __shared__ int cand[TP_CAND];                            // 4 * unit + entry
    const float *p = probs + (size_t)blockIdx.x * (size_t)ld_in;
    float *o = out + (size_t)blockIdx.x * (size_t)ld_out;
    const int t = threadIdx.x, n4 = tp_units<VEC>(V);
    // f(key) for every entry of the row.  Short loop bodies: 32 entries of a thread unrolled in registers were bound by the
    // fetch of instructions that a wavefront runs once (top-k 21 us against 16).
    auto each = [&](auto f) {
        constexpr int U = FITS || !VEC ? 2 : 4; // units in flight (of words: 2 x 4 loads)
        for (int i0 = t; i0 < n4; i0 += TP_THREADS * U) {
            f32x4 x[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int i = i0 + TP_THREADS * j;
                x[j] = i < n4 ? (FITS ? row[i] : tp_load4<VEC>(p, i, V)) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int j = 0; j < U; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) f(tp_key(x[j][e]));
        }
    };
    // The row is fetched (one that fits LDS: once); a top-k that looks for candidates finds each thread's largest entry on the way and looks at
    // one entry of every fourth unit of a thread for a weight.
    uint32_t sample = 0; // the key of one entry, the lanes' spread over the row: the first of one of the thread's own units
    auto take_sample = [&]() {
        const int own = t + TP_THREADS * ((t & 63) * ((n4 - t + TP_THREADS - 1) / TP_THREADS) >> 6);
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
        if (own < n4) {
            if constexpr (FITS || VEC) x = FITS ? row[own] : tp_load4<VEC>(p, own, V);
            else if (tp_entry<VEC>(own, 0) < V) x[0] = p[tp_entry<VEC>(own, 0)];
        }
        sample = tp_key(x[0]);
        return x;
    };
    float most = 0.f;
    int nz = 0; // of the wavefront's looks, those that found a weight
    if (FITS || (BY_COUNT && FRONT)) {
        for (int i0 = t & ~63; i0 < n4; i0 += TP_THREADS * 8) { // (the same bounds for a whole wavefront)
            f32x4 x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = tp_load4<VEC>(p, min(i0 + (t & 63) + TP_THREADS * j, n4 - 1), V);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int i = i0 + (t & 63) + TP_THREADS * j;
                if (FITS && i < n4) row[i] = x[j]; // (read back by the same thread; clear() below has the barrier for others)
                if (FRONT && BY_COUNT && j % 4 == 0) nz += __popcll(__ballot(i < n4 && x[j][j / 4] >= TP_LEAST));
                if (FRONT && BY_COUNT && i < n4) most = fmaxf(fmaxf(most, fmaxf(x[j][0], x[j][1])), fmaxf(x[j][2], x[j][3])); // (the same token at one thread only)
            }
        }
    }
    if (FRONT && BY_COUNT && (t & 63) == 0) sm_nz[t >> 6] = (uint8_t)min(nz, 255);
    auto unchanged = [&]() {
        for (int v = t; v < V; v += TP_THREADS) o[v] = p[v];
    };
    auto add_of = [](uint32_t key) { return BY_COUNT ? (Bin)1 : (Bin)tp_weight(key); };
    // The histogram of the row's entries with live(key), by bin(key).  Additions to one address are carried out one after another, and
    // the weights of a flat row are all in one bin (32000 equal ones: 116 us for the row, 16 for one of a softmax): each wavefront looks
    // at an entry per lane from all over the row, and where a quarter of those are in one bin it adds that bin's up in registers (43 us;
    // a vote at every entry took 20 - 40 % of the kernel).
    auto crowded_bin = [&](auto live, auto bin) { // (in front of clear(): most wavefronts wait at its barrier anyway)
        const bool l = live(sample);
        const unsigned long long lanes = __ballot(l);
        if (!lanes) return -1;
        const int b = bin(sample);
        const int first = __builtin_amdgcn_readlane(b, __ffsll((long long)lanes) - 1), last = __builtin_amdgcn_readlane(b, 63 - __clzll((long long)lanes));
        const int n1 = __popcll(__ballot(l && b == first)), n2 = __popcll(__ballot(l && b == last));
        return max(n1, n2) < 16 ? -1 : n1 >= n2 ? first : last;
    };
    auto histogram = [&](int hot, auto live, auto bin) {
        if (__builtin_expect(hot < 0, 1)) {
            each([&](uint32_t key) {
                if (live(key)) atomicAdd(&hist[bin(key)], add_of(key));
            });
        } else {
            unsigned long long sum = 0;
            each([&](uint32_t key) {
                if (live(key)) {
                    if (bin(key) == hot) sum += add_of(key);
                    else atomicAdd(&hist[bin(key)], add_of(key));
                }
            });
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) sum += shfl_xor_u64(sum, o);
            if ((t & 63) == 0) atomicAdd(&hist[hot], (Bin)sum);
        }
    };
    auto clear = [&]() {
        hist[t] = 0;
        hist[t + TP_THREADS] = 0;
        __syncthreads();
    };
    // the bin, from the top, in which the running sum reaches `need`; `need` becomes what it has to contribute, binw what it holds.
    // first: `need` comes from the total
    unsigned long long need = 0, target = 0, binw = 0, S = 0;
    auto choose = [&](bool first) -> int {
        __syncthreads();
        // thread t owns bins 2047 - 2t and 2046 - 2t, so thread order is descending weight order
        const unsigned long long a = hist[TP_BINS - 1 - 2 * t], b = hist[TP_BINS - 2 - 2 * t];
        unsigned long long total;
        const unsigned long long before = block_excl_scan(a + b, sm_wave, total);
        if (first) {
            S = total;
            if (BY_COUNT) {
                need = P24; // the k-th token of the order
            } else {
                // target = ceil(P24 * S / 2^24) from the 128-bit product, at least 1
                const unsigned long long lo = (unsigned long long)P24 * S, hi = __umul64hi((unsigned long long)P24, S);
                const unsigned long long lo2 = lo + 16777215ull, hi2 = hi + (lo2 < lo ? 1ull : 0ull);
                need = (hi2 << 40) | (lo2 >> 24);
                if (need < 1) need = 1;
            }
            target = need;
            if (S == 0 || need > S) return -1; // nothing has a weight; top-k: k reaches into the tokens without one
        }
        if (before < need && need <= before + a) {
            sm_bin = TP_BINS - 1 - 2 * t;
            sm_above = before;
            sm_binw = a;
        } else if (before + a < need && need <= before + a + b) {
            sm_bin = TP_BINS - 2 - 2 * t;
            sm_above = before + a;
            sm_binw = b;
        }
        __syncthreads();
        need -= sm_above;
        binw = sm_binw;
        const int bin = sm_bin;
        __syncthreads(); // everyone has read the choice before the next one overwrites it
        return bin;
    };

    if (t == 0) sm_n = sm_nc = 0;
    // Candidates, where few tokens have a weight (what a filter in front has left), or where the k-th largest of the threads' largest tokens
    // bounds the k-th of the row from below: the tokens of that bin and above, usually hardly more than k.  Histogram, boundary and sums
    // then take two entries per thread instead of 32 and more, and the row is written as zeros with the kept tokens put in.  Otherwise, and
    // where they turn out to be too many, everything below works on the row.  us, before -> now: 5 rows of 32000, top-k 40 15.3 -> 13.0, 200 16.2 ->
    // 14.5, top-p behind top-40 12.6 -> 9.2; of 50257 28.7 -> 19.4, 29.7 -> 21.2, 26.5 -> 12.0; 9 of 128256 41 -> 25, 42 -> 27.5, 38 -> 17.
    int nc = 0; // candidates (0: the row)
    auto gather = [&](float least) { // those of at least this probability
        for (int i0 = t; i0 < n4 && __hip_atomic_load(&sm_nc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <= TP_CAND; i0 += TP_THREADS * 2) {
            f32x4 x[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) x[j] = FITS ? row[min(i0 + TP_THREADS * j, n4 - 1)] : tp_load4<VEC>(p, min(i0 + TP_THREADS * j, n4 - 1), V);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (i0 + TP_THREADS * j < n4 && fmaxf(fmaxf(x[j][0], x[j][1]), fmaxf(x[j][2], x[j][3])) >= least) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (x[j][e] >= least) {
                            const int at = atomicAdd(&sm_nc, 1);
                            if (at < TP_CAND) {
                                cand[at] = 4 * (i0 + TP_THREADS * j) + e;
                                if (!FITS) reinterpret_cast<float *>(row)[at] = x[j][e];
                            }
                        }
                }
        }
        __syncthreads();
        const int n = __builtin_amdgcn_readfirstlane(sm_nc);
        nc = n <= TP_CAND && (!BY_COUNT || P24 <= (unsigned)n) ? n : 0;
    };
    auto candidate = [&](int i) { return reinterpret_cast<const float *>(row)[FITS ? cand[i] : i]; };
    auto each_candidate = [&](auto f) {
        for (int i = t; i < nc; i += TP_THREADS) f(tp_key(candidate(i)));
    };
    auto few_have_a_weight = [&](unsigned limit) { // by the wavefronts' counts, up to 255 each (more than the limit wherever a wavefront looks more often)
        const u32x4 c = *reinterpret_cast<const u32x4 *>(sm_nz);
        uint32_t n = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) n = __builtin_amdgcn_sad_u8(c[w], 0u, n); // + its four bytes
        return n <= limit;
    };
    const auto live = [](uint32_t key) { return key != 0; };
    const auto bin = [](uint32_t key) { return tp_bin(key); };
    int hot = -1;
    if constexpr (FRONT && BY_COUNT) {
        __syncthreads();
        float least = 0.f;
        const unsigned looks = n4 / (4 * TP_THREADS) * TP_THREADS + min(n4 % (4 * TP_THREADS), TP_THREADS);
        if (few_have_a_weight((unsigned)((unsigned long long)TP_CAND * looks / (unsigned)V))) {
            least = TP_LEAST;
        } else {
            clear();
            if (most >= TP_LEAST) atomicAdd(&hist[tp_bin(tp_key(most))], (Bin)1);
            const int b = choose(true);
            // (of threads with one above the bound; where they are most of them, so are the tokens above it - all those of a flat row)
            if (b >= 0 && P24 - need + binw <= TP_CAND / 2) least = u2f(tp_bin_prefix(b) << 17) * TP_LEAST;
        }
        if (least > 0.f) gather(least);
        if (!nc) {
            take_sample();
            hot = crowded_bin(live, bin);
        }
        clear();
    } else {
        // A top-p takes the histogram's samples for the look (of a longer row with 16-byte loads all four entries of their units: the limit is small
        // there) and adds the wavefronts' counts up behind the barrier that there is anyway.  Where nothing comes of it - every call that sets
        // top-p alone - it costs 0.1 - 0.2 us (5 rows, top-p 0.9, us, no look | a look of its own with a barrier of its own | now: 9001 entries 11.5 |
        // 11.9 | 11.7, 32000 18.8 | 19.2 | 18.9; top-p 0.3 of 128256 46.2 | 47.2 | 46.3, of 262144 87.2 | 88.9 | 87.2).
        const f32x4 x = take_sample();
        unsigned limit = 0;
        if constexpr (FRONT) {
            constexpr int LOOKS = !FITS && VEC ? 4 : 1;
            limit = TP_CAND * LOOKS * TP_THREADS / (unsigned)V;
            int n = 0;
#pragma unroll
            for (int e = 0; e < LOOKS; ++e) n += __popcll(__ballot(x[e] >= TP_LEAST));
            if ((t & 63) == 0) sm_nz[t >> 6] = (uint8_t)min(n, 255);
        }
        hot = crowded_bin(live, bin);
        clear();
        if (FRONT && __builtin_expect(few_have_a_weight(limit), 0)) gather(TP_LEAST);
    }
    if (nc) each_candidate([&](uint32_t key) { atomicAdd(&hist[bin(key)], add_of(key)); });
    else histogram(hot, live, bin);
    const int bin0 = choose(true);
    if (S == 0) { // nothing has a weight: the row is returned as it is
        unchanged();
        return;
    }
    uint32_t tau = 0;                  // key of the last kept token (0: top-k keeps every token with a weight and some without)
    unsigned long long n_ties, n_keep; // tokens of that weight, and how many of them are kept
    unsigned long long kept;           // weight of the kept set
    if (bin0 >= 0) {
        // the boundary bin's tokens to the list; top-k: the weight above the bin on the way
        uint32_t prefix = tp_bin_prefix(bin0);
        // more of them than the list holds, by what the bin holds and the largest weight in it (a flat row): no list
        const bool crowded = binw > (unsigned long long)TP_LIST * (BY_COUNT ? 1u : tp_weight((prefix << 17) | 0x1ffffu));
        unsigned long long above_w = 0;
        if (__builtin_expect(crowded, 0)) {
            if (BY_COUNT) {
                unsigned long long mine = 0;
                each([&](uint32_t key) { mine += (key >> 17) > prefix ? tp_weight(key) : 0u; });
                block_excl_scan(mine, sm_wave, above_w);
            }
        } else {
            unsigned long long mine = 0;
            const auto pick = [&](uint32_t key) {
                const uint32_t k17 = key >> 17;
                if (k17 >= prefix) {
                    if (k17 == prefix) {
                        const int at = atomicAdd(&sm_n, 1);
                        if (at < TP_LIST) list[at] = key;
                    } else if (BY_COUNT) {
                        mine += tp_weight(key);
                    }
                }
            };
            if (nc) each_candidate(pick);
            else each(pick);
            if (BY_COUNT) block_excl_scan(mine, sm_wave, above_w);
        }
        __syncthreads();
        const int n = crowded ? TP_LIST + 1 : sm_n;
        if (n <= TP_RANK) { // few: the token in whose turn the sum is reached finds itself
            if (t < n) {
                const uint32_t key = list[t];
                unsigned long long above = 0, equal = 0;
                for (int i = 0; i < n; ++i) {
                    const uint32_t other = list[i];
                    const unsigned long long add = add_of(other);
                    above += other > key ? add : 0ull;
                    equal += other == key ? add : 0ull;
                }
                if (above < need && need <= above + equal) { // (equal tokens write the same)
                    sm_bin = (int)key;
                    sm_above = above;
                    sm_binw = equal;
                }
            }
            __syncthreads();
            tau = (uint32_t)sm_bin;
            need -= sm_above;
            binw = sm_binw;
            __syncthreads();
        } else if (n <= TP_LIST && __syncthreads_and(list[t] == list[0] || t >= n) && __syncthreads_and(list[t + TP_THREADS] == list[0] || t + TP_THREADS >= n)) {
            tau = list[0]; // all of them equal
        } else { // the 17 bits behind the bin's, by digits
            for (int low = 17; low > 0;) {
                const int nb = low < 11 ? low : 11;
                const auto live = [&](uint32_t key) { return (key >> low) == prefix; };
                const auto digit = [&](uint32_t key) { return (int)((key >> (low - nb)) & ((1u << nb) - 1)); };
                const int hot = n <= TP_LIST ? -1 : crowded_bin(live, digit);
                clear();
                if (n <= TP_LIST) {
                    for (int i = t; i < n; i += TP_THREADS)
                        if (live(list[i])) atomicAdd(&hist[digit(list[i])], add_of(list[i]));
                } else {
                    histogram(hot, live, digit);
                }
                prefix = (prefix << nb) | (uint32_t)choose(false);
                low -= nb;
            }
            tau = prefix;
        }
        const unsigned long long w = tp_weight(tau);
        if (BY_COUNT) {
            n_ties = binw;
            n_keep = need;
        } else if (binw == w) { // one token of that weight, the usual case (two 64-bit divisions by 1024 threads take 2 us)
            n_ties = n_keep = 1;
        } else {
            n_ties = binw / w;
            n_keep = (need + w - 1) / w;
        }
        if (BY_COUNT) {
            // above the boundary inside the bin: summed over the list (or the row)
            unsigned long long in_bin = 0, more;
            const uint32_t first = tp_bin_prefix(bin0);
            if (n <= TP_LIST) {
                for (int i = t; i < n; i += TP_THREADS) in_bin += list[i] > tau ? tp_weight(list[i]) : 0u;
            } else {
                each([&](uint32_t key) {
                    if (key > tau && (key >> 17) == first) in_bin += tp_weight(key);
                });
            }
            block_excl_scan(in_bin, sm_wave, more);
            kept = above_w + more + n_keep * w;
        } else {
            kept = target - need + n_keep * w; // everything above tau (target - need) plus the kept tokens of weight tau
        }
    } else { // top-k past the tokens with a weight (S of them): all of those, and the first k - S of the others
        unsigned long long mine = 0;
        each([&](uint32_t key) { mine += tp_weight(key); });
        block_excl_scan(mine, sm_wave, kept);
        n_ties = (unsigned long long)V - S;
        n_keep = P24 - S;
    }
    int cut = V; // ties are kept up to and including this index
    if (__builtin_expect(n_keep < n_ties, 0)) {
        // the n_keep-th token of weight tau in index order: every wavefront counts a contiguous part of the row, and the one whose part holds it
        // looks for it there (a part per thread read a line per entry: 1 row of 128256 equal weights 159 us, now 110).  A part that one look
        // covers is looked at once, with as many loads as it has, and the sums in front of it are asked for together (5 rows of equal weights,
        // top-k 40, us, a part per thread | two looks of 16 loads and one sum after another | now: 1000 entries 11.3 | 12.7 | 11.0, 3001 17.4 |
        // 19.4 | 17.2, 6000 18.0 | 18.6 | 17.4).
        auto find_cut = [&](auto tu_, auto once_) {
            constexpr int TU = decltype(tu_)::value; // loads in flight
            constexpr bool ONCE = decltype(once_)::value; // a look covers the part
            const int lane = t & 63, wave = t >> 6;
            const int part = ((V + TP_WAVES - 1) / TP_WAVES + 63) & ~63, v0 = wave * part, v1 = min(v0 + part, V);
            auto ties = [&](int v, unsigned long long (&m)[TU]) { // of v .. v + 64 TU - 1
                float x[TU];
#pragma unroll
                for (int j = 0; j < TU; ++j) {
                    const int at = min(v + 64 * j + lane, V - 1);
                    if constexpr (FITS) x[j] = reinterpret_cast<const float *>(row)[VEC ? at : ((at >> 12) * TP_THREADS + (at & (TP_THREADS - 1))) * 4 + ((at >> 10) & 3)]; // (see tp_entry)
                    else x[j] = p[at];
                }
#pragma unroll
                for (int j = 0; j < TU; ++j) m[j] = __ballot(v + 64 * j + lane < v1 && tp_key(x[j]) == tau);
            };
            unsigned long long m[TU], cnt = 0, before = 0;
            for (int v = v0; ONCE || v < v1; v += 64 * TU) {
                ties(v, m);
#pragma unroll
                for (int j = 0; j < TU; ++j) cnt += __popcll(m[j]);
                if (ONCE) break;
            }
            __syncthreads(); // (sm_wave may still be read)
            if (lane == 0) sm_wave[wave] = cnt;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < TP_WAVES; ++w) before += w < wave ? sm_wave[w] : 0ull;
            if (before < n_keep && n_keep <= before + cnt) { // (one wavefront)
                bool found = false;
                for (int v = v0; v < v1 && !found; v += 64 * TU) {
                    if (!ONCE) ties(v, m);
#pragma unroll
                    for (int j = 0; j < TU; ++j) {
                        const unsigned long long c = __popcll(m[j]);
                        if (!found && before + c >= n_keep) {
                            found = true;
                            if ((m[j] >> lane & 1) && before + __popcll(m[j] & ((1ull << lane) - 1)) + 1 == n_keep) sm_cut = v + 64 * j + lane;
                        }
                        before += found ? 0 : c;
                    }
                }
            }
        };
        if (FITS && V <= 64 * 4 * TP_WAVES) find_cut(std::integral_constant<int, 4>{}, std::true_type{});
        else if (FITS && V <= 64 * 8 * TP_WAVES) find_cut(std::integral_constant<int, 8>{}, std::true_type{});
        else if (FITS && V <= 64 * 16 * TP_WAVES) find_cut(std::integral_constant<int, 16>{}, std::true_type{});
        else find_cut(std::integral_constant<int, 16>{}, std::false_type{});
        __syncthreads();
        cut = sm_cut;
    }
    const float Z = __fmul_rn(__ull2float_rn(kept), 2.3283064365386963e-10f), rZ = __fdiv_rn(1.0f, Z);
    if (nc) { // (nothing of the row is read any more: in place is fine)
        if (VEC) {
            for (int i = t; i < V / 4; i += TP_THREADS) *reinterpret_cast<f32x4 *>(o + 4 * i) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        for (int v = (VEC ? V / 4 * 4 : 0) + t; v < V; v += TP_THREADS) o[v] = 0.f;
        __syncthreads(); // the zeros are in front of what replaces them
        for (int i = t; i < nc; i += TP_THREADS) {
            const float x = candidate(i);
            const uint32_t key = tp_key(x);
            const int v = tp_entry<VEC>(cand[i] >> 2, cand[i] & 3);
            if (key > tau || (key == tau && v <= cut)) o[v] = key < 0x3f800000u || key >= 0x4f800000u ? __fdiv_rn(x, Z) : tp_divide(x, Z, rZ);
        }
        return;
    }
    constexpr int U = FITS || !VEC ? 2 : 4;
    for (int i0 = t; i0 < n4; i0 += TP_THREADS * U) {
        f32x4 x[U];
#pragma unroll
        for (int j = 0; j < U; ++j) { // (a thread reads what it writes: in place is fine)
            const int i = i0 + TP_THREADS * j;
            x[j] = i < n4 ? (FITS ? row[i] : tp_load4<VEC>(p, i, V)) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int i = i0 + TP_THREADS * j;
            f32x4 y;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t key = tp_key(x[j][e]);
                const bool keep = key > tau || (key == tau && tp_entry<VEC>(i, e) <= cut);
                float q = tp_divide(x[j][e], Z, rZ);
                if (keep && (key < 0x3f800000u || key >= 0x4f800000u)) q = __fdiv_rn(x[j][e], Z); // outside its range (a kept token without a weight, or of 1 and more)
                y[e] = keep ? q : 0.f;
            }
            if (VEC && 4 * i + 3 < V) {
                *reinterpret_cast<f32x4 *>(o + 4 * i) = y;
            } else if (i < n4) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (tp_entry<VEC>(i, e) < V) o[tp_entry<VEC>(i, e)] = y[e];
            }
        }
    }
}
template <bool BY_COUNT>
static void launch_filter(const float *probs, long long ld_in, int rows, int V, unsigned arg, float *out, long long ld_out, hipStream_t st) {
    if (rows <= 0) return;
    const bool vec = ((reinterpret_cast<uintptr_t>(probs) | reinterpret_cast<uintptr_t>(out)) & 15) == 0 && (rows == 1 || (ld_in % 4 == 0 && ld_out % 4 == 0));
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(rows), dim3(TP_THREADS), 0, st, probs, ld_in, V, arg, out, ld_out); };
    const bool front = BY_COUNT ? V >= TP_FRONT_K && arg <= TP_FEW : V >= TP_FRONT;
    auto pick = [&](auto v) {
        constexpr bool VEC = decltype(v)::value;
        if (V <= TP_FITS) {
            if (front) go(top_p_filter_kernel<BY_COUNT, VEC, true, true>);
            else go(top_p_filter_kernel<BY_COUNT, VEC, true, false>);
        } else {
            if (front) go(top_p_filter_kernel<BY_COUNT, VEC, false, true>);
            else go(top_p_filter_kernel<BY_COUNT, VEC, false, false>);
        }
    };
    if (vec) pick(std::true_type{});
    else pick(std::false_type{});
}
void launch_top_p_filter(const float *probs, long long ld_in, int rows, int V, unsigned P24, float *out, long long ld_out, hipStream_t st) {
    launch_filter<false>(probs, ld_in, rows, V, P24, out, ld_out, st);
}
void launch_top_k_filter(const float *probs, long long ld_in, int rows, int V, int k, float *out, long long ld_out, hipStream_t st) {
    launch_filter<true>(probs, ld_in, rows, V, (unsigned)k, out, ld_out, st);
}

// ------------------------------------------------------------------ sampling / argmax of plain rows

__global__ __launch_bounds__(SAMPLE_THREADS) void sample_rows_kernel(const float *probs, int64_t ld, int V, const float *u,
                                                                     int32_t *token_out) {
    __shared__ unsigned long long sm_wave[SAMPLE_WAVES];
    __shared__ int sm_tok;
    __shared__ float sm_val[SAMPLE_WAVES];
    __shared__ int sm_idx[SAMPLE_WAVES];
    const int b = blockIdx.x;
    RowSrc P;
    P.row = probs + (size_t)b * ld;
    P.from_logits = 0;
    P.inv_t = 1.f;
    P.mx = 0.f;
    P.invZ = 1.f;
    int tok = block_inv_cdf<false>(P, P, V, 0, V, false, 0, u[b], sm_wave, &sm_tok);
    if (tok < 0) tok = block_argmax(P, V, sm_val, sm_idx);
    if (threadIdx.x == 0) token_out[b] = tok;
}
void launch_sample_rows(const float *probs, int64_t ld, int B, int V, const float *u, int32_t *token_out,
                        hipStream_t st) {
    if (B <= 0) return;
    hipLaunchKernelGGL(sample_rows_kernel, dim3(B), dim3(SAMPLE_THREADS), 0, st, probs, ld, V, u, token_out);
}

// Softmax of a row and one token from it in one launch, for short rows of one statistics segment (no workgroup waits for another):
// the statistics, the probabilities and the token are those of the three launches it replaces, bit for bit (the first two by
// the same operations in the same order, the token because the inverse CDF adds integers).  The row is read three times, twice
// from the caches, by one workgroup, so the launches saved pay up to some length only.  A draft's call of one fp32 layer, 1 | 16
// sequences, us, three launches -> this one: 1024 logits 38.1 -> 35.5 | 41.4 -> 37.8, 4096 42.8 -> 38.7 | 45.4 -> 42.0, 6000 44.5 -> 41.2 |
// 47.4 -> 45.6, 8192 44.4 -> 43.7 | 47.3 -> 48.1, 12288 48.7 -> 51.6 | 52.1 -> 57.4, 16384 49.0 -> 55.5 | 54.0 -> 63.3.
constexpr int SOFTMAX_SAMPLE_MAX = 6144;
static_assert(SOFTMAX_SAMPLE_MAX <= STATS_SEG, "one statistics segment");
__global__ __launch_bounds__(256) void softmax_sample_kernel(const float *logits, int V, float inv_t, float *probs, int64_t ld, const float *u,
                                                             int32_t *token_out) {
    __shared__ unsigned long long sm_wave[4];
    __shared__ int sm_tok;
    __shared__ float sm_val[4];
    __shared__ int sm_idx[4];
    __shared__ float2 sm_stats;
    const int b = blockIdx.x;
    const float *x = logits + (size_t)b * V;
    float *p = probs + (size_t)b * ld;
    const float2 r = segment_stats(x, V, inv_t, (V % 4 == 0) && ((reinterpret_cast<uintptr_t>(x) & 15) == 0));
    if (threadIdx.x == 0) sm_stats = r;
    __syncthreads();
    RowSrc P;
    P.row = x;
    P.from_logits = 1;
    P.inv_t = inv_t;
    P.mx = sm_stats.x;
    P.invZ = inv_norm(sm_stats.y);
    for (int v = threadIdx.x; v < V; v += 256) p[v] = P.at(v);
    int tok = block_inv_cdf<false, 4>(P, P, V, 0, V, false, 0, u[b], sm_wave, &sm_tok);
    if (tok < 0) tok = block_argmax(P, V, sm_val, sm_idx);
    if (threadIdx.x == 0) token_out[b] = tok;
}
bool launch_softmax_sample(const float *logits, int B, int V, float inv_t, float *probs, int64_t ld, const float *u, int32_t *token_out, hipStream_t st) {
    if (V > SOFTMAX_SAMPLE_MAX) return false;
    if (B > 0) hipLaunchKernelGGL(softmax_sample_kernel, dim3(B), dim3(256), 0, st, logits, V, inv_t, probs, ld, u, token_out);
    return true;
}

// Running argmax: the lowest index on ties; NaNs lose to everything, -inf included (nothing but NaNs: NO_INDEX, which loses in turn
// when pieces of a row meet)
constexpr int NO_INDEX = 0x7fffffff;
struct Argmax {
    float best = -INFINITY;
    int index = NO_INDEX;
    __device__ __forceinline__ void see(float v, int i) {
        if (v > best || (v == best && i < index)) {
            best = v;
            index = i;
        }
    }
    __device__ __forceinline__ int token() const { return index == NO_INDEX ? 0 : index; }
};
// (value, index) of the largest of x[0 .. n), indices from `first`.  ARGMAX_UNROLL independent loads per thread are in flight: a row
// is read once and the kernel is bound by how many loads a compute unit has outstanding.  Valid in thread 0.
constexpr int ARGMAX_UNROLL = 8;
template <int THREADS> __device__ __forceinline__ Argmax block_argmax_range(const float *x, int n, int first) {
    Argmax a;
    if ((reinterpret_cast<uintptr_t>(x) & 15) == 0) {
        const f32x4 *x4 = reinterpret_cast<const f32x4 *>(x);
        const int n4 = n / 4;
        for (int i0 = threadIdx.x; i0 < n4; i0 += THREADS * ARGMAX_UNROLL) {
            f32x4 t[ARGMAX_UNROLL];
#pragma unroll
            for (int j = 0; j < ARGMAX_UNROLL; ++j) t[j] = x4[min(i0 + THREADS * j, n4 - 1)]; // (past the end: the last unit again, with its own index)
#pragma unroll
            for (int j = 0; j < ARGMAX_UNROLL; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) a.see(t[j][e], 4 * min(i0 + THREADS * j, n4 - 1) + e);
        }
        if ((int)threadIdx.x < n - 4 * n4) a.see(x[4 * n4 + threadIdx.x], 4 * n4 + threadIdx.x);
    } else {
        for (int i0 = threadIdx.x; i0 < n; i0 += THREADS * ARGMAX_UNROLL) {
            float t[ARGMAX_UNROLL];
#pragma unroll
            for (int j = 0; j < ARGMAX_UNROLL; ++j) t[j] = x[min(i0 + THREADS * j, n - 1)];
#pragma unroll
            for (int j = 0; j < ARGMAX_UNROLL; ++j) a.see(t[j], min(i0 + THREADS * j, n - 1));
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float b2 = __shfl_xor(a.best, o);
        const int i2 = __shfl_xor(a.index, o);
        a.see(b2, i2);
    }
    __shared__ float sm_val[THREADS / 64];
    __shared__ int sm_idx[THREADS / 64];
    if ((threadIdx.x & 63) == 0) {
        sm_val[threadIdx.x >> 6] = a.best;
        sm_idx[threadIdx.x >> 6] = a.index;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < THREADS / 64; ++w) a.see(sm_val[w], sm_idx[w]);
        if (a.index != NO_INDEX) a.index += first;
    }
    return a;
}

// one workgroup per row (a draft's call has one to a few rows, and a second launch that merges segments costs 4.5 us:
// 32000 logits 12.9 -> 6 us with the loads in flight together)
__global__ __launch_bounds__(SAMPLE_THREADS) void argmax_rows_kernel(const float *x, int64_t ld, int V, int32_t *out) {
    const Argmax a = block_argmax_range<SAMPLE_THREADS>(x + (size_t)blockIdx.x * ld, V, 0);
    if (threadIdx.x == 0) out[blockIdx.x] = a.token();
}
void launch_argmax_rows(const float *logits, int64_t ld, int B, int V, int32_t *token_out, hipStream_t st) {
    if (B <= 0) return;
    hipLaunchKernelGGL(argmax_rows_kernel, dim3(B), dim3(SAMPLE_THREADS), 0, st, logits, ld, V, token_out);
}

// Greedy: accept while the draft token is the target row's argmax; next = argmax at the first mismatch.  The rows are cut into
// segments (grid: segments x rows) whose (value, index) pairs the second launch, which scans the positions anyway, merges in
// index order: one workgroup per row left a row's stream to one compute unit (72 rows of 128256 logits: 45.6 us = 0.8 TB/s).
__global__ __launch_bounds__(256) void argmax_segment_kernel(const float *x, int V, int seg_len, float2 *part) {
    const int r0 = blockIdx.x * seg_len;
    const Argmax a = block_argmax_range<256>(x + (size_t)blockIdx.y * V + r0, min(seg_len, V - r0), r0);
    if (threadIdx.x == 0) part[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = make_float2(a.best, __int_as_float(a.index));
}
constexpr int GREEDY_SEGS = 16; // most segments of a row
// one wavefront per sequence, lane i = position i (K + 1 <= 16 positions)
// row_argmax: the rows' tokens where they were not cut (part NULL)
__global__ __launch_bounds__(64) void greedy_finish_kernel(const float2 *part, int nseg, const int32_t *row_argmax, const int32_t *draft, int K,
                                                           int32_t *n_accepted, int32_t *next_token) {
    const int b = blockIdx.x, i = min((int)threadIdx.x, K);
    const size_t row = (size_t)b * (K + 1) + i;
    int tok;
    if (part) {
        Argmax a;
        float2 p[GREEDY_SEGS];
#pragma unroll
        for (int s = 0; s < GREEDY_SEGS; ++s) p[s] = part[row * nseg + min(s, nseg - 1)]; // (all asked for together; the last one again past the end)
#pragma unroll
        for (int s = 0; s < GREEDY_SEGS; ++s) a.see(p[s].x, __float_as_int(p[s].y));
        tok = a.token();
    } else {
        tok = row_argmax[row];
    }
    const bool mismatch = (int)threadIdx.x >= K || draft[(size_t)b * K + threadIdx.x] != tok;
    const int n = min(__ffsll((long long)__ballot(mismatch)) - 1, K);
    if ((int)threadIdx.x == n) {
        n_accepted[b] = n;
        next_token[b] = tok;
    }
}
// segments per row: at most GREEDY_SEGS, of at least 4096 entries each while that fills the chip (2048 workgroups), and no more than the
// workspace holds pairs for (avail: bytes)
static int greedy_segments(int64_t rows, int V, size_t avail, int &seg_len) {
    int64_t nseg = std::min<int64_t>(std::min<int64_t>(GREEDY_SEGS, V / 4096), 2048 / rows);
    nseg = std::max<int64_t>(1, std::min<int64_t>(nseg, (int64_t)(avail / (sizeof(float2) * (size_t)rows))));
    seg_len = (int)((V + nseg - 1) / nseg);
    seg_len = (seg_len + 3) & ~3; // keeps the 16-byte alignment of an aligned row
    return (V + seg_len - 1) / seg_len;
}
void launch_greedy_accept(const float *p_logits, const int32_t *draft, int B, int K, int V, void *scratch, size_t scratch_bytes,
                          int32_t *n_accepted, int32_t *next_token, hipStream_t st) {
    if (B <= 0) return;
    const int64_t rows = (int64_t)B * (K + 1);
    int seg_len;
    const int nseg = greedy_segments(rows, V, scratch_bytes, seg_len);
    if (nseg == 1) { // (a row's one workgroup needs no pair)
        launch_argmax_rows(p_logits, V, (int)rows, V, (int32_t *)scratch, st);
        hipLaunchKernelGGL(greedy_finish_kernel, dim3(B), dim3(64), 0, st, (const float2 *)nullptr, 1, (const int32_t *)scratch, draft, K, n_accepted, next_token);
        return;
    }
    hipLaunchKernelGGL(argmax_segment_kernel, dim3(nseg, (unsigned)rows), dim3(256), 0, st, p_logits, V, seg_len, (float2 *)scratch); // (rows <= 1024 here)
    hipLaunchKernelGGL(greedy_finish_kernel, dim3(B), dim3(64), 0, st, (const float2 *)scratch, nseg, (const int32_t *)nullptr, draft, K, n_accepted, next_token);
}

} // namespace ss
