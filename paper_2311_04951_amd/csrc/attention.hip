// Multi-query-row causal decode attention against the contiguous KV cache ("attention" in Section 3's
// cost breakdown; the cache is the one of Sections 2 and 4.2).
//
// For sequence b, head h, the M = K+1 new rows (row i at absolute position L_b + i) attend cache
// positions 0..L_b + i; the rows' own keys/values were appended before this kernel runs, so everything
// is read back from the cache.  The KV range is split over workgroups (grid.x) and, inside a
// workgroup, over 4 wavefronts; every key/value tile is read from HBM exactly once and serves all M
// rows: the M query rows are the 16-wide B operand of the MFMAs (held in registers), keys and
// (block-transposed) values are the streamed A operand, 16 bytes per lane.
//
//   S^T[pos][m]  = sum_e K[pos][e] * Q[m][e]        (keys as A, queries as B)
//   O^T[e][m]   += sum_pos V^T[e][pos] * P[m][pos]  (transposed values as A, softmax weights as B)
//
// The row order of a key tile is permuted so that the score registers a lane receives are exactly
// the 8 (bf16) or 4 (f32) consecutive positions it must supply as the B operand of the P.V product:
// tile t, row i  <->  position p0 + (i/4)*E + 4t + (i%4).
// Online softmax in the log2 domain per wave; waves, then splits, are merged by log-sum-exp in a
// fixed order.  The second kernel merges the splits, normalises and writes the result as the
// activation planes the O projection consumes.
#include <type_traits>
#include "attention_core.h"

namespace ss {

// merge over splits, normalise, write activation planes: grid (R, H), block HD
template <typename T, int HD>
__global__ __launch_bounds__(256) void attn_partial_kernel(AttnArgs a) {
    __shared__ AttnSmem<HD, 4> sm;
    attn_unit<T, HD, 4>(a, blockIdx.x, blockIdx.y, blockIdx.z, a.len[blockIdx.z], sm);
}

// a single split: the workgroup normalises and writes the activation planes itself (no partials, no merge launch)
template <typename T, int HD, int NWX = 4>
__global__ __launch_bounds__(NWX * 64) void attn_direct_kernel(AttnArgs a) {
    __shared__ AttnSmem<HD, NWX> sm;
    attn_unit<T, HD, NWX, false, true>(a, 0, blockIdx.y, blockIdx.z, a.len[blockIdx.z], sm);
}

// A single split of many positions, bf16: blocks of 64 positions go round the wavefronts, each block's keys, then its values, through the
// wavefront's own 16 KB of LDS.  What bounds it is the cache's bytes: keys and values of a block are 16 KB in one piece each, so every
// load-to-LDS instruction brings a contiguous kilobyte, where loads in operand layout take half lines of 16 rows.  The other wavefronts' requests
// fill the time in which one multiplies (a compute unit has some 32 KB of loads in flight; 64 KB or more are asked for).
//   A layer, us, loads in operand layout -> blocks -> and the non-temporal bit (when: streams_kv in api.hip): 7B shape 8 x 9 rows at 2000 | 4000 positions
// 189.6 -> 188.4 -> 178.0 | 235.6 -> 233.9 -> 215.1; 9 sequences (288 units, 32 compute units with two) 321 -> 298 -> 278 at 4000.
template <int HD, int NW>
__global__ __launch_bounds__(NW * 64) void attn_blocks_kernel(AttnArgs a) {
    typedef bf16_t T;
    constexpr int NKC = HD / 32, NDT = HD / 16, BLOCK = 64 * HD * 2, UPR = HD / 8, RPI = 64 / UPR; // (16-byte units of a key, keys per load instruction)
    static_assert(sizeof(AttnSmem<HD, NW>) <= NW * BLOCK, "");
    __shared__ __align__(16) unsigned char lds[NW * BLOCK];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int h = blockIdx.y, b = blockIdx.z, L = a.len[b], ntot = min(L + a.M, a.chunk); // (the host's bound on the lengths, which fits the cache)
    unsigned char *buf = lds + wave * BLOCK;
    const uint32_t to = lds_address(buf);

    ActPlanes<T> qp{const_cast<T *>(reinterpret_cast<const T *>(a.q)), a.q_plane, a.ldq};
    const int qrow = min(b * a.M + c, a.R - 1);
    Act<T> q[NKC];
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) q[kc] = load_act(qp, (size_t)qrow * a.ldq + h * HD + kc * 32 + g * 8);
    const char *Kb = reinterpret_cast<const char *>(a.kcache) + ((size_t)b * a.H + h) * a.S * HD * 2;
    const char *Vb = reinterpret_cast<const char *>(a.vcache) + ((size_t)b * a.H + h) * a.S * HD * 2;

    // Unit u of key r sits at position u xor (r mod 4 + 4 (r / 8 mod 4 or 2)): the sixteen keys of a tile (below) in different banks.  Values:
    // unit u of head element e at u xor (e mod 8).
    const uint32_t voff = (uint32_t)(lane / 8) * 128u + (uint32_t)((lane & 7) ^ (lane >> 3)) * 16u;
    auto request = [&](const char *p, auto offset) {
        if (a.stream) {
#pragma unroll
            for (int i = 0; i < BLOCK / 1024; ++i) dma16<true>(p + i * 1024, offset(i), to + i * 1024);
        } else {
#pragma unroll
            for (int i = 0; i < BLOCK / 1024; ++i) dma16(p + i * 1024, offset(i), to + i * 1024);
        }
    };
    auto request_keys = [&](int blk) {
        request(Kb + (size_t)blk * BLOCK, [&](int i) {
            const int r = i * RPI + lane / UPR, f = (r & 3) + 4 * ((r >> 3) & (UPR / 4 - 1)); // key of the block
            return (uint32_t)(lane / UPR) * HD * 2u + (uint32_t)((lane % UPR) ^ f) * 16u;
        });
    };
    auto request_values = [&](int blk) { request(Vb + (size_t)blk * BLOCK, [&](int) { return voff; }); };
    const bool row_ok = c < a.M;
    const int row_limit = L + c; // last position row c may attend
    float m_run = NEG_BIG, l_run = 0.f;
    f32x4 o[NDT];
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (wave * 64 < ntot) request_keys(wave);
    for (int blk = wave; blk * 64 < ntot; blk += NW) {
        wait_vmcnt_at_most<0>();
        asm volatile("" ::: "memory");
        // keys of a half block's tile t: row i is position 8 (i / 4) + 4t + i mod 4, so that lane (c, g) receives 8g + 4t + v
        f32x4 s[2][2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                s[hh][t] = f32x4{0.f, 0.f, 0.f, 0.f};
                const int r = 32 * hh + (c >> 2) * 8 + 4 * t + (c & 3), f = (c & 3) + 4 * ((c >> 2) & (UPR / 4 - 1));
#pragma unroll
                for (int kc = 0; kc < NKC; ++kc) s[hh][t] = mma(s[hh][t], *reinterpret_cast<const u32x4 *>(buf + r * HD * 2 + ((kc * 4 + g) ^ f) * 16), q[kc]);
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the keys have been read
        request_values(blk);
        float pv[2][8], bm = NEG_BIG;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int pos = blk * 64 + 32 * hh + g * 8 + e;
                const float x = row_ok && pos <= row_limit ? s[hh][e >> 2][e & 3] * a.scale_log2e : NEG_BIG;
                pv[hh][e] = x;
                bm = fmaxf(bm, x);
            }
        bm = fmaxf(bm, __shfl_xor(bm, 16));
        bm = fmaxf(bm, __shfl_xor(bm, 32));
        const float m_new = fmaxf(m_run, bm), alpha = exp2f(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float p = pv[hh][e] > 0.5f * NEG_BIG ? exp2f(pv[hh][e] - m_new) : 0.f;
                l_run += p;
                pv[hh][e] = p;
            }
        m_run = m_new;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) o[dt] *= alpha;
        const Act<T> P[2] = {pack_act(pv[0], T{}), pack_act(pv[1], T{})};
        wait_vmcnt_at_most<0>();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            if (hh && blk * 64 + 32 >= ntot) break; // (what lies there may be no numbers, which a weight of zero would not undo; up to 31 positions of the half before it are multiplied, as in attn_unit)
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt)
                o[dt] = mma(o[dt], *reinterpret_cast<const u32x4 *>(buf + (dt * 16 + c) * 128 + ((hh * 4 + g) ^ (c & 7)) * 16), P[hh]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // ... and the values
        if ((blk + NW) * 64 < ntot) request_keys(blk + NW);
    }
    // The wavefronts' results, merged in order as attn_unit does.  (Code of its own: as a function that both call it changed the registers and the first
    // loads of every kernel that attn_unit is in, 0.2 - 0.35 us a layer of few rows.)
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    auto &sm = *reinterpret_cast<AttnSmem<HD, NW> *>(lds);
    __syncthreads(); // nobody reads keys or values any more
    if (g == 0) {
        sm.m[wave][c] = m_run;
        sm.l[wave][c] = l_run;
    }
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int v = 0; v < 4; ++v) sm.o[wave][dt][v][lane] = o[dt][v];
    __syncthreads();
    if (!row_ok) return;
    float mstar = sm.m[0][c], wt[NW], l = 0.f;
#pragma unroll
    for (int w = 1; w < NW; ++w) mstar = fmaxf(mstar, sm.m[w][c]);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        wt[w] = exp2f(sm.m[w][c] - mstar);
        l += sm.l[w][c] * wt[w];
    }
    ActPlanes<T> out{reinterpret_cast<T *>(a.act_out), a.act_out_plane, a.ld_out};
    for (int dt = wave; dt < NDT; dt += NW)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float acc = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) acc += sm.o[w][dt][v][lane] * wt[w];
            store_act(out, (size_t)(b * a.M + c) * a.ld_out + h * HD + dt * 16 + 4 * g + v, acc / l);
        }
}

template <typename T>
__global__ void attn_merge_kernel(AttnArgs a) {
    const int row = blockIdx.x, h = blockIdx.y, e = threadIdx.x;
    ActPlanes<T> out{reinterpret_cast<T *>(a.act_out), a.act_out_plane, a.ld_out};
    store_act(out, (size_t)row * a.ld_out + h * a.hd + e, attn_merge_elem<false>(a, row, h, e));
}

template <typename T> static void launch_attention_t(const AttnArgs &a, hipStream_t st) {
    dim3 grid(a.nsplit, a.H, a.B);
    if (a.nsplit == 1) {
        if constexpr (std::is_same<T, bf16_t>::value) {
            // From 256 positions on (four blocks); a call has one split of so many from 256 units on.  A layer at 250 | 400 positions, us, attn_direct_kernel ->
            // blocks: 7B shape, 16 sequences of one row 107.9 -> 108.3 | 113.6 -> 115.7, 8 x 9 rows 142.6 -> 142.7 | 144.6 -> 144.1, 16 x 16
            // 259.5 -> 260.1 | 271.5 -> 273.5; 13B shape, 10 x 9 260 -> 250 | 262 -> 255.  Heads of 128: eight wavefronts, 128 KB of LDS, are no faster than four
            // where a compute unit has one unit (8 x 9 rows at 520 | 4000 positions 147.0 | 218.7 with eight, 147.7 | 215.1 with four; at lengths from
            // 3188 to 4080 218.1, 214.5) and keep a second one out where it has two (16 x 16 at 400 276, 273).
            if (a.chunk >= 256 && a.hd >= 64) {
                if (a.hd == 128) hipLaunchKernelGGL((attn_blocks_kernel<128, 4>), grid, dim3(256), 0, st, a);
                else hipLaunchKernelGGL((attn_blocks_kernel<64, 8>), grid, dim3(512), 0, st, a);
                return;
            }
        }
        // few units with a short context (one split by the host's choice): 8 waves, so that a wave has one step up to 256 positions
        if (a.hd == 128 && a.B * a.H < 256) {
            hipLaunchKernelGGL((attn_direct_kernel<T, 128, 8>), grid, dim3(512), 0, st, a);
            return;
        }
        if (a.hd == 128) hipLaunchKernelGGL((attn_direct_kernel<T, 128>), grid, dim3(256), 0, st, a);
        else if (a.hd == 64) hipLaunchKernelGGL((attn_direct_kernel<T, 64>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((attn_direct_kernel<T, 32>), grid, dim3(256), 0, st, a);
        return;
    }
    if (a.hd == 128) hipLaunchKernelGGL((attn_partial_kernel<T, 128>), grid, dim3(256), 0, st, a);
    else if (a.hd == 64) hipLaunchKernelGGL((attn_partial_kernel<T, 64>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((attn_partial_kernel<T, 32>), grid, dim3(256), 0, st, a);
    hipLaunchKernelGGL((attn_merge_kernel<T>), dim3(a.R, a.H), dim3(a.hd), 0, st, a);
}

void launch_attention(int dtype, const AttnArgs &a, hipStream_t st) {
    if (dtype) launch_attention_t<bf16_t>(a, st);
    else launch_attention_t<float>(a, st);
}

} // namespace ss
