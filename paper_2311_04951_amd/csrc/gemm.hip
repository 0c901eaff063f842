// Weight-streaming skinny GEMM for the "linear layers" of the verify pass (Section 3: K+1 rows are
// evaluated together, and the pass is bound by reading the weights once).
//
//   out[m][n] = sum_k act[m][k] * W[n][k],   W row-major [N][K]; the R rows form row tiles of 16, and a
//   workgroup multiplies every weight chunk it streams with up to RT row tiles (weights are read once for
//   up to 16*RT rows).
//
// At most 16 rows (gemm_cols_kernel): the output columns (pairs of them for the fused epilogues) are dealt out evenly over the compute
// units.  Weights and activation rows (packed planes) come through LDS by load-to-LDS instructions that take whole 128-byte lines, into a
// ring of the wavefront's own, and are read back as the A and B operands of the MFMAs.  The waves interleave over K in 128-byte steps,
// their partial tiles are summed in a fixed order through LDS (deterministic), two columns of a row per thread, and finished:
//   STORE   plain fp32 store (LM head)
//   RESID   h += ...            (O projection, down projection)
//   SWIGLU  silu(gate) * up     (gate and up columns in one workgroup) -> activation planes
//   QKV     rotary embedding of q and k (pairs j, j + hd/2 in one workgroup), q -> activation
//           planes, k and v -> KV cache at positions len[b] + i
#include <type_traits>
#include "ss_device.h"
#include "ss_kernels.h"

namespace ss {

// What an epilogue reads besides the sums (the residual, the sequence's length and the rotary factors), for V columns of a row: a
// kernel whose K loop takes many memory round trips asks for them behind its first request, so that the epilogue adds none.
template <int V> struct EpiPre {
    float resid[V];
    float2 rope[V];
    int len;       // of the row's sequence
    float gain[V]; // deferred norm, producer: the next norm's gains of these columns
};

// Where columns sit.  `col`: the first of them, for EPI_QKV the weight row of the first one in the first half of its head
// ((head over [q heads | k heads | v heads]) * head_dim + column in the head).
struct QkvPlace {
    int region, h, j0; // 0 q, 1 k, 2 v; head; column in the head
};
__device__ __forceinline__ QkvPlace qkv_place(const GemmArgs &a, int col) {
    const int hh = col >> (31 - __clz(a.hd)); // head_dim is 32, 64 or 128
    const int region = (hh >= a.H) + (hh >= 2 * a.H);
    return QkvPlace{region, hh - region * a.H, col & (a.hd - 1)};
}
// cache position of row m whose sequence holds `len` (host validation keeps it inside; the bounds are a second one)
__device__ __forceinline__ int qkv_position(const GemmArgs &a, int m, int len) { return min(len + m - m / a.M * a.M, min(a.max_pos, a.S) - 1); }
template <int EPI, int V> __device__ __forceinline__ void epi_prefetch(const GemmArgs &a, int m, int col, EpiPre<V> &pre) {
    m = min(m, a.R - 1); // a row past the end asks for the last row's operands and never uses them
    if constexpr (EPI == EPI_RESID) {
        const size_t o0 = (size_t)m * a.ldo + col;
        if (col + V <= a.N && a.ldo % V == 0 && (reinterpret_cast<uintptr_t>(a.resid) & (4 * V - 1)) == 0) {
            typedef float vec __attribute__((ext_vector_type(V)));
            const vec r = *reinterpret_cast<const vec *>(a.resid + o0);
#pragma unroll
            for (int v = 0; v < V; ++v) pre.resid[v] = r[v];
        } else {
#pragma unroll
            for (int v = 0; v < V; ++v) pre.resid[v] = a.resid[(size_t)m * a.ldo + min(col + v, a.N - 1)];
        }
        if (a.nsq_out) {
#pragma unroll
            for (int v = 0; v < V; ++v) pre.gain[v] = a.norm_gain[min(col + v, a.N - 1)];
        }
    } else if constexpr (EPI == EPI_QKV) {
        pre.len = a.len[m / a.M];
    }
}
// ... what depends on the first: the rotary factors of the row's position
template <int EPI, int V> __device__ __forceinline__ void epi_prefetch_rope(const GemmArgs &a, int m, int col, EpiPre<V> &pre) {
    if constexpr (EPI == EPI_QKV) {
        const QkvPlace at = qkv_place(a, col);
        if (at.region < 2) {
            const float2 *p = a.rope + (size_t)qkv_position(a, min(m, a.R - 1), pre.len) * (a.hd / 2) + at.j0;
#pragma unroll
            for (int v = 0; v < V; ++v) pre.rope[v] = p[v];
        }
    }
}

// The lengths of the cache move with the last projection of a pass: by the first wave of the first workgroup.
template <int EPI> __device__ __forceinline__ void move_lengths(const GemmArgs &a) {
    if constexpr (EPI == EPI_RESID) {
        if (a.len_add && (blockIdx.x | blockIdx.y | blockIdx.z) == 0 && threadIdx.x < 64)
            for (int b = threadIdx.x; b < a.len_batch; b += 64) a.len_add[b] += a.len_delta;
    }
}

// Rotary embedding and stores of V column pairs (j0 + v, j0 + hd/2 + v) of row m.
template <typename T, int V>
__device__ __forceinline__ void qkv_store(const GemmArgs &a, int m, const QkvPlace &at, float (&x0)[V], float (&x1)[V], int pos, const float2 (&rope)[V]) {
    const int b = m / a.M, h = at.h, j0 = at.j0;
    if (at.region < 2) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const float2 cs = rope[v];
            const float p0 = x0[v] * cs.x - x1[v] * cs.y;
            const float p1 = x0[v] * cs.y + x1[v] * cs.x;
            x0[v] = p0;
            x1[v] = p1;
        }
    }
    if (at.region == 0) {
        ActPlanes<T> q{reinterpret_cast<T *>(a.act_out), a.act_out_plane, a.ld_act_out};
        const size_t o = (size_t)m * a.ld_act_out + h * a.hd + j0;
        store_act_cols(q, o, x0, V);
        store_act_cols(q, o + a.hd / 2, x1, V);
    } else if (at.region == 1) {
        T *kc = reinterpret_cast<T *>(a.kcache) + (((size_t)b * a.H + h) * a.S + pos) * a.hd + j0;
        store_cols(kc, x0); // (the cache is 16-byte aligned, j0 a multiple of V)
        store_cols(kc + a.hd / 2, x1);
    } else {
        // values are kept transposed inside blocks of 64 positions: [pos/64][hd][64]
        T *vc = reinterpret_cast<T *>(a.vcache) + ((size_t)b * a.H + h) * a.S * a.hd + ((size_t)(pos >> 6) * a.hd) * 64 + (pos & 63);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            vc[(size_t)(j0 + v) * 64] = to_storage<T>(x0[v]);
            vc[(size_t)(j0 + a.hd / 2 + v) * 64] = to_storage<T>(x1[v]);
        }
    }
}

// Epilogue of V columns from `col` (see qkv_place) of row m < R: x0, and x1 the second half of a fused pair; pre: operands
// fetched ahead by epi_prefetch for this row and these columns.  Returns, where a deferred norm is asked for, the sum of squares of
// the row's new values.
template <typename T, int EPI, int V>
__device__ __forceinline__ float epilogue_cols(const GemmArgs &a, int m, int col, float (&x0)[V], float (&x1)[V], const EpiPre<V> &pre) {
    if constexpr (EPI == EPI_STORE || EPI == EPI_RESID) {
        if constexpr (EPI == EPI_RESID) {
#pragma unroll
            for (int v = 0; v < V; ++v) x0[v] = pre.resid[v] + x0[v];
        }
        const size_t o0 = (size_t)m * a.ldo + col;
        if (col + V <= a.N && a.ldo % V == 0 && (reinterpret_cast<uintptr_t>(a.out) & (4 * V - 1)) == 0) {
            store_cols(a.out + o0, x0);
        } else {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                if (col + v < a.N) a.out[o0 + v] = x0[v];
                else x0[v] = 0.f;
            }
        }
        if (EPI == EPI_RESID && a.nsq_out) { // deferred norm: h * gain as planes
            ActPlanes<T> np{reinterpret_cast<T *>(a.norm_act), a.norm_act_plane, a.norm_ld};
            float y[V], sq = 0.f;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                y[v] = x0[v] * pre.gain[v];
                sq += x0[v] * x0[v];
            }
            store_act_cols(np, (size_t)m * a.norm_ld + col, y, a.N - col);
            return sq;
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
        ActPlanes<T> z{reinterpret_cast<T *>(a.act_out), a.act_out_plane, a.ld_act_out};
        float y[V];
#pragma unroll
        for (int v = 0; v < V; ++v) y[v] = x0[v] / (1.0f + expf(-x0[v])) * x1[v];
        store_act_cols(z, (size_t)m * a.ld_act_out + col, y, a.N - col);
    } else { // EPI_QKV
        qkv_store<T, V>(a, m, qkv_place(a, col), x0, x1, qkv_position(a, m, pre.len), pre.rope);
    }
    return 0.f;
}
// ... with the operands read here
template <typename T, int EPI, int V>
__device__ __forceinline__ void epilogue_cols(const GemmArgs &a, int m, int col, float (&x0)[V], float (&x1)[V]) {
    EpiPre<V> pre;
    epi_prefetch<EPI, V>(a, m, col, pre);
    epi_prefetch_rope<EPI, V>(a, m, col, pre);
    epilogue_cols<T, EPI, V>(a, m, col, x0, x1, pre);
}
// Epilogue of one output tile by one wave: lane (c, g) holds r[t][v] = the value of row m = rt*16 + c, column n0[t] + 4g + v.
template <typename T, int EPI>
__device__ __forceinline__ void apply_epilogue(const GemmArgs &a, float (&r)[(EPI == EPI_SWIGLU || EPI == EPI_QKV) ? 2 : 1][4],
                                               const int (&n0)[(EPI == EPI_SWIGLU || EPI == EPI_QKV) ? 2 : 1], int rt) {
    const int lane = threadIdx.x & 63, m = rt * 16 + (lane & 15);
    constexpr int LAST = (EPI == EPI_SWIGLU || EPI == EPI_QKV) ? 1 : 0;
    if (m < a.R) epilogue_cols<T, EPI, 4>(a, m, n0[0] + 4 * (lane >> 4), r[0], r[LAST]);
}

// The K steps of a workgroup in rotated order: step i of nst becomes (i + rot) mod nst; steps past the end stay there
// (they are masked).  The offset depends on the workgroup alone, so a tile's sum is always formed in the same order.
// (The golden ratio's multiples spread neighbours over K; a remainder would cost a division in front of the first load.)
__device__ __forceinline__ int k_rotation(int nst) { return (int)__umulhi(blockIdx.x * 0x9E3779B9u, (unsigned)nst); }
__device__ __forceinline__ int rotated(int i, int rot, int nst) {
    if (i >= nst) return i;
    i += rot;
    return i >= nst ? i - nst : i;
}

// Waits until at most n loads are in flight, LO <= n <= HI (n is the same for the wavefront).
template <int LO, int HI> __device__ __forceinline__ void wait_vmcnt(int n) {
    if constexpr (LO < HI) {
        if (n < HI) return wait_vmcnt<LO, HI - 1>(n);
    }
    wait_vmcnt_at_most<HI>();
}
// Waits until at most `loads` + FIXED loads are in flight (1 <= loads <= MOST).
template <int FIXED, int MOST> __device__ __forceinline__ void wait_for_step(int loads) {
    if constexpr (MOST > 1) {
        if (loads < MOST) return wait_for_step<FIXED, MOST - 1>(loads);
    }
    wait_vmcnt_at_most<FIXED + MOST>();
}

// Activations of the kernels for at most 16 rows, through a wave-private piece of LDS.  A step of a wave is UPS units
// of 16 bytes of K for every row and plane: PL * R * UPS pieces.  Loaded per lane into MFMA operand layout that is
// 2 * PL * UPS / 8 load instructions with R / 16 of their lanes active; instead ceil(PL * R * UPS / 64) full-width
// load-to-LDS instructions bring them (lane l of instruction i brings piece 64 i + l; the pieces land in lane order,
// 16 bytes each) and the operands are read back from LDS.  Piece (plane * R + row) * UPS + (unit xor row) holds unit
// `unit` of the row, so that the 16 rows a wave reads together fall into different banks.  Lanes of rows that do not
// exist read a slot that holds zeros.  Measured on the 7B-shaped layer: 5-row pass 3.62 -> 3.37 ms, 1 row 3.29 -> 3.18.
// (The plane is part of a piece's 32-bit offset: calls of at most 16 rows pack their planes 16 rows apart.)
template <typename T, int UPS, int RCAP = 16> struct ActStage { // RCAP: most rows (5, 8 or 16)
    static constexpr int PL = Traits<T>::PLANES, EPU = 16 / (int)sizeof(T);
    static constexpr int NDMA = (PL * RCAP * UPS + 63) / 64; // instructions that bring a step at RCAP rows
    static constexpr int SLOTS = NDMA * 64;                   // ... and the slots they fill
    static constexpr int BYTES = (SLOTS + 1) * 16; // LDS of one step of one wave (the last slot holds zeros)
    uint32_t off[NDMA]; // byte offset in the planes of this lane's piece of instruction i in the step at K = 0
    int ucol[NDMA];     // its first K element inside the step
    const char *base;
    int rows, npiece, kmax;

    // K: reduction length (a multiple of EPU)
    __device__ __forceinline__ void init(const GemmArgs &a, int K, int lane) {
        rows = min(a.R, RCAP);
        npiece = PL * rows * UPS;
        kmax = K - EPU;
        base = reinterpret_cast<const char *>(a.act);
#pragma unroll
        for (int i = 0; i < NDMA; ++i) {
            const unsigned p = min(i * 64 + lane, npiece - 1); // surplus lanes repeat the last piece into slots nobody reads
            const bool low = PL == 2 && p >= (unsigned)(rows * UPS);
            const unsigned rem = low ? p - rows * UPS : p, row = rem / UPS, pos = rem % UPS; // (UPS is a power of two)
            ucol[i] = (pos ^ (row & (UPS - 1))) * EPU;
            off[i] = ((low ? (uint32_t)a.act_plane : 0u) + row * (uint32_t)a.ld_act + ucol[i]) * (uint32_t)sizeof(T);
        }
    }
    __device__ __forceinline__ static void clear(unsigned char *region, int lane) {
        if (lane == 0) *reinterpret_cast<u32x4 *>(region + SLOTS * 16) = zero16();
    }
    __device__ __forceinline__ int loads() const { return (npiece + 63) / 64; } // instructions of a step
    // asks for the step that starts at K element k0, to LDS address `to`.  tail: the step ends inside its units: columns past the end
    // are clamped to the row's last unit (the weights there are zero, so any finite value does)
    __device__ __forceinline__ void request(uint32_t to, int k0, bool tail) const {
        const char *b = base + (size_t)k0 * sizeof(T);
        if (tail) {
#pragma unroll
            for (int i = 0; i < NDMA; ++i)
                if (i * 64 < npiece) dma16(b, off[i] - (uint32_t)(max(k0 + ucol[i] - kmax, 0) * (int)sizeof(T)), to + i * 1024);
            return;
        }
#pragma unroll
        for (int i = 0; i < NDMA; ++i)
            if (i * 64 < npiece) dma16(b, off[i], to + i * 1024);
    }
    // byte offset in a step's region of row c's unit `unit` of plane pl
    __device__ __forceinline__ int operand_offset(int c, int unit, int pl) const {
        return c < rows ? ((pl * rows + c) * UPS + (unit ^ (c & (UPS - 1)))) * 16 : SLOTS * 16;
    }
};
// A wavefront's n steps of K through a ring of NB (one or two) buffers of its own.  request(i, buffer) asks for its i-th step, use(i, buffer)
// multiplies it; between them the step's loads are waited for - with two buffers by wait_ahead(), which leaves the next step's in
// flight.  behind_first() runs behind the first request; what it asks for is older than the second step and has arrived when the first
// has.  with_first() runs then, and uses it.  (The compiler does not count the requests, which are assembly, and puts a vmcnt(0) of its own in
// front of the first such use: with two buffers the wavefronts that finish the launch wait for their second step there.)
template <int NB, class Request, class Use, class Wait, class Behind, class With>
__device__ __forceinline__ void ring_walk(int n, Request request, Use use, Wait wait_ahead, Behind behind_first, With with_first) {
    static_assert(NB == 1 || NB == 2, "a third buffer made every launch slower: no counted wait for two steps");
    if (n > 0) request(0, 0);
    behind_first();
    for (int i = 0, buf = 0; i < n; ++i) {
        const bool ahead = NB == 2 && i + 1 < n;
        if (ahead) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // what was read from the buffer that is filled now has arrived
            request(i + 1, buf ^ 1);
            wait_ahead();
        } else {
            wait_vmcnt_at_most<0>();
        }
        asm volatile("" ::: "memory");
        use(i, buf);
        if (i == 0) with_first();
        if (NB == 1 && i + 1 < n) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            request(i + 1, 0);
        }
        if (NB == 2) buf ^= 1;
    }
    if (n <= 0) with_first();
}

// Sum over the PS (4, 8 or 16) neighbouring lanes that share a row; every one of them gets it.
template <int PS> __device__ __forceinline__ float row_sum(float x) {
    auto add = [](float v, auto ctrl) { return v + u2f((uint32_t)__builtin_amdgcn_update_dpp(0, (int)f2u(v), decltype(ctrl)::value, 0xf, 0xf, true)); };
    x = add(x, std::integral_constant<int, 0xB1>{});  // quad_perm: lane xor 1
    x = add(x, std::integral_constant<int, 0x4E>{});  // quad_perm: lane xor 2
    if constexpr (PS >= 8) x = add(x, std::integral_constant<int, 0x141>{});  // row_half_mirror: the other four of eight
    if constexpr (PS >= 16) x = add(x, std::integral_constant<int, 0x140>{}); // row_mirror: the other eight of sixteen
    return x;
}

// int8 entries as bf16 (exact)
__device__ __forceinline__ uint32_t w8_pair_to_bf16x2(uint32_t x, int first_byte) {
    const float f0 = (float)((int)(x << (24 - 8 * first_byte)) >> 24); // sign-extended bytes
    const float f1 = (float)((int)(x << (16 - 8 * first_byte)) >> 24);
    return __builtin_amdgcn_perm(f2u(f1), f2u(f0), 0x07060302u); // |q| <= 127: the low 16 bits of the fp32 are zero
}
__device__ __forceinline__ u32x4 w8_to_bf16x8(uint32_t a, uint32_t b) {
    return u32x4{w8_pair_to_bf16x2(a, 0), w8_pair_to_bf16x2(a, 2), w8_pair_to_bf16x2(b, 0), w8_pair_to_bf16x2(b, 2)};
}

// int4 entries as bf16 values q / 16 (exact): dword j of a unit holds entries 8j .. 8j + 7, entry e in bits 4e .. 4e + 3, two's complement.  The
// conversion instruction takes the low four bits of a byte that it selects itself and makes a sixteenth of them: 13 instructions a
// dword (22 by shifts and integer conversions).
__device__ __forceinline__ u32x4 w4_to_bf16x8_sixteenths(uint32_t x) {
    uint32_t y = x >> 4;
    asm("" : "+v"(y)); // (one shift for all odd entries, not one each)
    uint32_t r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float f0 = __builtin_amdgcn_cvt_off_f32_i4((int)(x >> (8 * i) & 0xff)), f1 = __builtin_amdgcn_cvt_off_f32_i4((int)(y >> (8 * i) & 0xff));
        r[i] = __builtin_amdgcn_perm(f2u(f1), f2u(f0), 0x07060302u); // the low 16 bits of the fp32 are zero
    }
    return u32x4{r[0], r[1], r[2], r[3]};
}

// The same eight entries as bf16 values q + 136 (even entries: 0x4300 | n is 128 + n) and q + 24 (odd ones: 0x4180 | n << 3 is 16 + n; n the
// entry with its sign bit flipped, q + 8), without a conversion instruction: a byte permute places a byte in both halves of a register,
// for the upper half shifted right by one, so that its upper nibble lies where bf16 has a step of one there, and one three-operand
// logical instruction masks the nibbles, flips their signs and sets the exponents.  Nine vector instructions per eight entries (22 by
// conversions, 12 with both nibbles in the same place); the caller starts its sums at -(136, 24) * the activations (W4_BIAS).
__device__ __forceinline__ u32x4 w4_to_bf16x8_biased(uint32_t x) {
    const uint32_t y = x >> 1;
    uint32_t r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) // bytes [x.i, 0, y.i, 0] (selector bytes 0-3: second operand, 4-7: first, 0x0c: zero)
        r[i] = (__builtin_amdgcn_perm(y, x, 0x0c000c00u | ((4u + i) << 16) | (uint32_t)i) & 0x0078000Fu) ^ 0x41C04308u;
    return u32x4{r[0], r[1], r[2], r[3]};
}
constexpr uint32_t W4_BIAS = 0xC1C0C308u; // -136 and -24 as a pair of bf16

// The kernel for at most 16 rows, for every kind of matrix (QB: 0 storage type, 8 int8 with one scale per weight row, 4 int4 with one
// scale per 128 K entries).  blockIdx.x owns a share of the output columns, in quads of four (a quad of pairs for the fused epilogues:
// its first and its second half): the launcher deals them out evenly, so that every compute unit has the same number of bytes to
// fetch - with 16 columns to a workgroup the compute units with one workgroup more than the others were what a launch took (a 13B-shaped
// down projection, 320 workgroups on 256 units: 21 us the median workgroup, 37 the launch) - and stages the activations once for all
// its columns.  The NW wavefronts interleave over K in steps of 128 bytes of every row, each through a ring of NB buffers of its own;
// EI load instructions of eight weight rows (per half) make a step.  The 16-column tiles are cut from the first halves' rows and the second
// ones' behind them, so that an odd EI wastes at most one half tile, not one a half (a 7B-shaped QKV share is 24 + 24 rows: three tiles).
//   Up to 8 rows (RCAP), two planes: operand columns 0 .. 7 hold the rows' high parts and 8 .. 15 the low ones, one MFMA and one LDS read
// per k-block instead of two; the two halves of the sums are added in front of the epilogue.
//   int8: a lane's 16-byte unit holds 16 entries of its weight row, two k-blocks: lane (c, g) supplies k = 64h + 16g + 8j .. + 7 of the
// step to block (h, j) and reads the activations of exactly those; the row scale multiplies the finished sum.  int4: a unit holds 32
// entries, four k-blocks, all in scale group h of the step's two; a group accumulates into a fresh tile, which is added to the
// running sum times the group's scales of the lane's four columns (stored group-major, scale[group][column]).
//   Weights through LDS: a load-to-LDS instruction takes whole 128-byte lines of 8 rows (lane l: unit (l & 7) xor (row & 7) of row
// l >> 3), loads in operand layout would take half lines of 16.
//   In front of the first request stands only what it needs, and a lane finishes two columns of a row: a launch spent 0.6 - 1.3 us ahead
// of its first load and as much behind its last one.
//   Measured against 16 columns to a workgroup (us a launch, back to back, 5 rows; QKV, O, gate/up, down): 7B shape bf16 20.0, 9.0, 29.4, 18.2 ->
// 17.7, 7.9, 28.8, 16.5 (6.2 TB/s in gate/up); 13B 28.8, 16.0, 49.0, 35.4 -> 26.9, 11.3, 45.7, 24.3; 3B 15.6, 7.2, 17.9, 12.1 -> 11.8, 6.3, 17.7, 10.9;
// 7B int8 15.7, 7.8, 20.0, 14.3 -> 12.0, 6.3, 18.5, 11.7; int4 13.0, 7.2, 16.3, 11.2 -> 10.7, 5.9, 14.5, 9.7.  Heads of 32000 columns, K 4096: bf16
// 42.0 -> 40.6, int8 35.3 -> 24.0, int4 24.6 -> 17.2; 12 rows: gate/up 32.6 -> 31.2, 13B 59.0 -> 49.0, bf16 head 65.4 -> 43.3.
//   int4 and int8 launches were bound by vector instructions as much as by bytes (7B int4 gate/up: 387 a wavefront and step, 7.7 of its 14.5 us):
// the nine-instruction unpacking, sums that start at the biases' share, the packed tiles and a uniform branch for the ragged last step, five
// rows, 7B shape: 8 int4 layers 400 -> 380 us, 4 int8 layers 235 -> 228; 13B int4 at 8 rows, 3 layers 230 -> 222.
template <typename T, int QB, int EPI, int NW, int NB, int EI, int RCAP>
__global__ __launch_bounds__(NW * 64) void gemm_cols_kernel(GemmArgs a) {
    constexpr int E = Traits<T>::E, KB = 4 * E;
    constexpr int NH = (EPI == EPI_SWIGLU || EPI == EPI_QKV) ? 2 : 1, NT = (NH * EI + 1) / 2; // halves; 16-column tiles: the first halves' columns, then the second ones'
    constexpr bool HL = Traits<T>::PLANES == 2 && RCAP <= 8; // high and low rows side by side in one operand
    constexpr int SK = QB == 4 ? 256 : QB == 8 ? 128 : 128 / (int)sizeof(T); // K entries of a step
    constexpr int PV = HL ? 1 : Traits<T>::PLANES;
    constexpr int SW = QB == 4 ? (2 * NT * 16 + 63) / 64 : 0; // int4: load instructions for a step's scales
    typedef ActStage<T, SK * (int)sizeof(T) / 16, RCAP> Stage;
    constexpr int SBASE = NH * EI * 1024, WBYTES = SBASE + SW * 256, SBYTES = WBYTES + Stage::BYTES; // (the rows that an odd EI's last tile does not have read what follows)
    __shared__ __align__(16) unsigned char lds[NW][NB][SBYTES];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int K = a.K;

    // the workgroup's quads; weight rows of a column (of its first half)
    const int q0 = (int)blockIdx.x * a.quads + min((int)blockIdx.x, a.quads_rest), nq = a.quads + ((int)blockIdx.x < a.quads_rest ? 1 : 0);
    const int nrows_w = EPI == EPI_SWIGLU ? 2 * a.N : a.N;
    const int columns = EPI == EPI_QKV ? a.N / 2 : a.N;
    auto row_of = [&](int p) { // QKV: column p of the first halves is column p mod (hd / 2) of head p / (hd / 2)
        if constexpr (EPI == EPI_QKV) return p + (p & ~(a.hd / 2 - 1));
        else return p;
    };
    const size_t row_bytes = QB == 4 ? (size_t)K / 2 : QB == 8 ? (size_t)K : (size_t)K * sizeof(T);
    const int half_rows = EPI == EPI_QKV ? a.hd / 2 : a.N; // from a first half's row to its second half's
    const int wub = ((lane & 7) ^ (lane >> 3)) * 16;       // this lane's bytes of a step
    const int row0 = row_of(4 * q0);
    uint32_t woff[EI];
#pragma unroll
    for (int i = 0; i < EI; ++i) { // instruction i: rows 8i .. 8i + 7; columns that the workgroup or the matrix does not have repeat its last one
        const int r = min(8 * i + (lane >> 3), 4 * nq - 1);
        woff[i] = (uint32_t)((row_of(min(4 * q0 + r, columns - 1)) - row0) * (int)row_bytes) + wub;
    }
    const char *wbase = reinterpret_cast<const char *>(a.W) + (size_t)row0 * row_bytes;
    uint32_t soff[SW ? SW : 1]; // int4: word 64 i + lane of a step's scales is group h * 16 NT + column of the tiles
    bool sh[SW ? SW : 1];
#pragma unroll
    for (int i = 0; i < SW; ++i) {
        const int w = i * 64 + lane, hf = w % (16 * NT) / (8 * EI) % NH, r = w % (16 * NT) - hf * 8 * EI;
        sh[i] = w / (16 * NT) == 1;
        soff[i] = (uint32_t)(row_of(min(4 * q0 + min(r, 4 * nq - 1), columns - 1)) + hf * half_rows) * 4u;
    }
    // Every workgroup starts at another place of K and wraps around (k_rotation): with all of them walking K in step,
    // the loads of a moment differ by multiples of the row stride and meet in the same memory channels, and all ask
    // for the same activation lines (measured on the 7B-shaped layer: 6 % of the 5-row pass, QKV 33.3 -> 29.7 us).
    const int nst = (K + SK - 1) / SK;
    const int rot = k_rotation(nst);
    const bool ragged = K % SK != 0; // the last step ends inside its 128 bytes
    Stage stage;
    const uint32_t lds0 = lds_address(lds[wave][0]);

    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    int rdw[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) rdw[j] = (c * 8 + ((4 * j + g) ^ (c & 7))) * 16;
    auto read_act = [&](const unsigned char *cur, int unit, u32x4 (&av)[PV]) {
#pragma unroll
        for (int pl = 0; pl < PV; ++pl)
            av[pl] = *reinterpret_cast<const u32x4 *>(cur + WBYTES + (HL ? stage.operand_offset(c & 7, unit, c >> 3) : stage.operand_offset(c, unit, pl)));
    };
    auto mul = [&](f32x4 s, u32x4 w, const u32x4 (&av)[PV]) {
        if constexpr (Traits<T>::PLANES == 2) {
#pragma unroll
            for (int pl = 0; pl < PV; ++pl) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, av[pl]), s, 0, 0, 0);
            return s;
        } else {
            Act<T> b;
            b.p[0] = av[0];
            return mma(s, w, b);
        }
    };

    // The epilogue: thread i of the first EW wavefronts finishes columns 2 (i mod PS) and + 1 of row i / PS; what it needs besides the
    // sums is asked for behind the first step's request: operands of the epilogue, int8 scales, a deferred norm's sums of squares.
    constexpr int PS = EI == 1 ? 4 : EI == 2 ? 8 : 16, EW = ((HL ? 8 : 16) * PS + 63) / 64, NSQ4 = NSQ_MAX_PARTS / 4 / PS;
    static_assert(EW <= NW && EI <= 4 && NW * NB * SBYTES <= 160 * 1024, "");
    const int er = (int)threadIdx.x / PS, ep = (int)threadIdx.x % PS; // row, column pair
    const int m = er, col = row_of(min(4 * q0 + min(2 * ep, 4 * nq - 2), (columns - 1) & ~1));
    const bool ends = wave < EW;
    EpiPre<2> pre;
    float wsc[NH][2], rs = 1.0f;
    float4 nsq[NSQ4];

    const int n = wave < nst ? (nst - wave + NW - 1) / NW : 0;
    ring_walk<NB>(
        n,
        [&](int i, int buf) {
            const int st = rotated(wave + i * NW, rot, nst);
            const bool tail = ragged && st == nst - 1;
            const uint32_t to = lds0 + buf * SBYTES;
            const uint32_t over = tail ? (uint32_t)max(st * 128 + wub - ((int)row_bytes - 16), 0) : 0u; // past a ragged end: the row's last unit, zeroed after the read (int4: a whole group, skipped)
            const char *b = wbase + (size_t)st * 128;
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
                for (int j = 0; j < EI; ++j) dma16<true>(b + (h ? half_rows * row_bytes : 0), woff[j] - over, to + (h * EI + j) * 1024);
#pragma unroll
            for (int j = 0; j < SW; ++j) dma4(a.wscale + (size_t)(2 * st) * nrows_w, soff[j] + (sh[j] && !tail ? (uint32_t)nrows_w * 4u : 0u), to + SBASE + j * 256);
            if (i == 0) { // (nothing of it stands in front of the first weights' request)
                int l = lane;
                asm volatile("" : "+v"(l));
                stage.init(a, K, l);
            }
            stage.request(to + WBYTES, st * SK, tail);
        },
        [&](int i, int buf) {
            const unsigned char *cur = lds[wave][buf];
            const int st = ragged || QB == 4 ? rotated(wave + i * NW, rot, nst) : 0;
            auto read_w = [&](int t, int j) { return *reinterpret_cast<const u32x4 *>(cur + t * 2048 + rdw[j]); };
            if constexpr (QB == 0) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    u32x4 w[NT], av[PV];
#pragma unroll
                    for (int t = 0; t < NT; ++t) w[t] = read_w(t, j);
                    read_act(cur, 4 * j + g, av);
                    if (ragged && (2 * st + j) * KB + g * E >= K) {
#pragma unroll
                        for (int t = 0; t < NT; ++t) w[t] = zero16();
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[t] = mul(acc[t], w[t], av);
                }
            } else if constexpr (QB == 8) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    u32x4 w[NT], av[2][PV];
#pragma unroll
                    for (int t = 0; t < NT; ++t) w[t] = read_w(t, h);
#pragma unroll
                    for (int j = 0; j < 2; ++j) read_act(cur, 8 * h + 2 * g + j, av[j]);
                    if (ragged && st * SK + 64 * h + 16 * g >= K) {
#pragma unroll
                        for (int t = 0; t < NT; ++t) w[t] = zero16();
                    }
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int t = 0; t < NT; ++t) acc[t] = mul(acc[t], w8_to_bf16x8(w[t][2 * j], w[t][2 * j + 1]), av[j]);
                }
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (2 * st + h < K / 128) { // (the same for the whole wave)
                        u32x4 av[4][PV];
#pragma unroll
                        for (int j = 0; j < 4; ++j) read_act(cur, 16 * h + 4 * g + j, av[j]);
                        // what the biases of the entries add to the group's sums, off them (the same for every output column)
                        f32x4 start = f32x4{0.f, 0.f, 0.f, 0.f};
                        const u32x4 bias = u32x4{W4_BIAS, W4_BIAS, W4_BIAS, W4_BIAS};
#pragma unroll
                        for (int j = 0; j < 4; ++j) start = mul(start, bias, av[j]);
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            const u32x4 w = read_w(t, h);
                            const f32x4 sc = *reinterpret_cast<const f32x4 *>(cur + SBASE + ((h * NT + t) * 16 + 4 * g) * 4);
                            f32x4 part = start;
#pragma unroll
                            for (int j = 0; j < 4; ++j) part = mul(part, w4_to_bf16x8_biased(w[j]), av[j]);
#pragma unroll
                            for (int v = 0; v < 4; ++v) acc[t][v] += sc[v] * part[v];
                        }
                    }
                }
            }
        },
        [&] { wait_for_step<NH * EI + SW, Stage::NDMA>(stage.loads()); },
        [&] {
#pragma unroll
            for (int s = 0; s < NB; ++s) Stage::clear(lds[wave][s] + WBYTES, lane);
            if (!ends) return;
            epi_prefetch<EPI, 2>(a, m, col, pre);
            if constexpr (QB == 8) {
#pragma unroll
                for (int h = 0; h < NH; ++h)
#pragma unroll
                    for (int v = 0; v < 2; ++v) wsc[h][v] = a.wscale[min(col + h * half_rows + v, nrows_w - 1)];
            }
            if (a.act_nsq) { // the row's PS threads read its partial sums, 16 bytes at a time in turn
                const float4 *p = reinterpret_cast<const float4 *>(a.act_nsq + (size_t)min(m, a.R - 1) * a.act_nsq_parts);
#pragma unroll
                for (int i = 0; i < NSQ4; ++i) nsq[i] = p[min(ep + i * PS, a.act_nsq_parts / 4 - 1)]; // (surplus slots repeat the last one and are not added)
            }
        },
        [&] {
            if (!ends) return;
            epi_prefetch_rope<EPI, 2>(a, m, col, pre);
            if (a.act_nsq) { // the row scale of a deferred norm on the activations
                float s = 0.f;
#pragma unroll
                for (int i = 0; i < NSQ4; ++i) s += ep + i * PS < a.act_nsq_parts / 4 ? (nsq[i].x + nsq[i].y) + (nsq[i].z + nsq[i].w) : 0.f;
                rs = 1.0f / sqrtf(row_sum<PS>(s) / (float)K + a.norm_eps);
            }
        });

    // the waves' partial tiles, each in the wavefront's own ring (nothing lands there any more), summed in order by the epilogue's threads
    static_assert(NT * 1024 <= SBYTES, "");
#pragma unroll
    for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4 *>(lds[wave][0] + (t * 64 + lane) * 16) = acc[t];
    __syncthreads();
    move_lengths<EPI>(a);
    if (!ends) return;
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    float x[NH][2];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        // column 2 ep of half h, row r of the tiles: tile r / 16, lane group (r / 4) mod 4, accumulator registers r mod 4 and + 1
        const int r = h * 8 * EI + 2 * ep, at = r / 16 * 1024 + ((r / 4 & 3) * 16 + (er & 15)) * 16 + (r & 3) * 4;
        f32x2 sum = *reinterpret_cast<const f32x2 *>(lds[0][0] + at);
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += *reinterpret_cast<const f32x2 *>(lds[w][0] + at);
        if constexpr (HL) { // + the sums of the low parts (row + 8)
            f32x2 low = *reinterpret_cast<const f32x2 *>(lds[0][0] + at + 128);
#pragma unroll
            for (int w = 1; w < NW; ++w) low += *reinterpret_cast<const f32x2 *>(lds[w][0] + at + 128);
            sum += low;
        }
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            x[h][v] = sum[v];
            if constexpr (QB == 8) x[h][v] *= wsc[h][v];
            x[h][v] *= rs; // (1 without a deferred norm: exact)
        }
    }
    float sq = 0.f;
    if (m < a.R && ep < 2 * nq && 4 * q0 + 2 * ep < columns) sq = epilogue_cols<T, EPI, 2>(a, m, col, x[0], x[NH - 1], pre);
    if (EPI == EPI_RESID && a.nsq_out) { // deferred norm: the row's sum of squares over the workgroup's columns
        sq = row_sum<PS>(sq);
        if (ep == 0 && m < a.R) a.nsq_out[(size_t)m * a.nsq_parts + blockIdx.x] = sq;
    }
}

// More than 16 rows of fp32 models (bf16 and quantised matrices: gemm_tile_kernel): the waves of a workgroup split the output columns instead
// of K, so that all of them walk K together and share the activation rows through LDS - with R rows
// the activations a wave needs are R*4/32 times its weight bytes, too much to fetch per wave from L2.
//   * wave w owns the 16 (or, fused epilogues, 2 x 16) weight rows of tile blockIdx.x*NW + w and the
//     complete K sum of its outputs: no reduction across waves;
//   * K is walked in slabs of 256 bytes per row.  The slab of all RT*16 rows goes from memory straight
//     into LDS (global_load_lds, no registers), two steps ahead of its use, into one of three buffers;
//     a 1 KB load instruction carries four rows, and the 16-byte units of a row are stored at position
//     (unit ^ row) so that the 16 rows a wave reads together hit different banks without padding;
//   * three weight slabs per wave in registers (one being multiplied, two in flight).
// Every step issues the same number of memory instructions (addresses are clamped into the operands; weights
// past K are zeroed after the load, so whatever finite activation sits there contributes nothing): the
// waits on "the loads issued two steps ago" are exact counts.
constexpr int WIDE_SLAB_BYTES = 256; // bytes of K per row and slab

// acc0 / acc1 += one weight chunk x one activation k-block, into two independent accumulators
__device__ __forceinline__ void mma_split(f32x4 &acc0, f32x4 &acc1, u32x4 w, const Act<float> &b, int kb) {
    if (kb & 1) acc1 = mma(acc1, w, b);
    else acc0 = mma(acc0, w, b);
}

__device__ __forceinline__ void wide_barrier() { // workgroup barrier that orders LDS traffic only (no vmcnt(0))
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
}
// columns of wave tile `tile`: n0[t] = first column of its t-th 16-column output tile; returns the number of wave tiles
template <int EPI>
__device__ __forceinline__ int wide_tile_cols(const GemmArgs &a, int tile, int (&n0)[(EPI == EPI_SWIGLU || EPI == EPI_QKV) ? 2 : 1]) {
    int ntiles;
    if constexpr (EPI == EPI_QKV) {
        const int per_head = a.hd / 32;
        ntiles = 3 * a.H * per_head;
        const int tl = min(tile, ntiles - 1);
        const int hh = tl / per_head; // head index over [q heads | k heads | v heads]
        n0[0] = hh * a.hd + (tl % per_head) * 16;
        n0[1] = n0[0] + a.hd / 2;
    } else if constexpr (EPI == EPI_SWIGLU) {
        ntiles = (a.N + 15) / 16;
        n0[0] = min(tile, ntiles - 1) * 16;
        n0[1] = a.N + n0[0];
    } else {
        ntiles = (a.N + 15) / 16;
        n0[0] = min(tile, ntiles - 1) * 16;
    }
    return ntiles;
}
// split-K partial tiles: [split][wave tile][row tile][t][v][lane] fp32, i.e. the accumulator layout of a wave
__device__ __forceinline__ size_t splitk_index(int z, int ntiles, int tile, int row_tiles, int rt, int NT, int t, int v, int lane) {
    return (((((size_t)z * ntiles + tile) * row_tiles + rt) * NT + t) * 4 + v) * 64 + lane;
}

template <int EPI, int NW, int RT>
__global__ __launch_bounds__(NW * 64) void gemm_wide_kernel(GemmArgs a) {
    typedef float T;
    constexpr int E = Traits<T>::E, KB = 4 * E;
    constexpr int NT = (EPI == EPI_SWIGLU || EPI == EPI_QKV) ? 2 : 1;
    constexpr int WIDE_KS = WIDE_SLAB_BYTES / (int)sizeof(T); // elements of K per slab
    constexpr int KBS = WIDE_KS / KB;                         // k-blocks per slab (4)
    constexpr int EPU = 16 / (int)sizeof(T);                  // elements per 16-byte unit
    constexpr int ROWS = RT * 16;
    constexpr int BUF = ROWS * WIDE_SLAB_BYTES;               // bytes of one slab buffer
    constexpr int GROUPS = ROWS / 4;                          // 1 KB load instructions per slab (4 rows each)
    constexpr int DPW = (GROUPS + NW - 1) / NW;               // ... per wave
    constexpr int WN = NT * KBS;                              // weight loads per wave and step
    __shared__ __align__(16) unsigned char slab0[BUF], slab1[BUF], slab2[BUF];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 15, g = lane >> 4;
    const int rt0 = blockIdx.y * RT;
    const int K = a.K;
    const int tile = blockIdx.x * NW + wave;

    int n0[NT];
    const int ntiles = wide_tile_cols<EPI>(a, tile, n0);
    const bool tile_live = tile < ntiles; // a dead wave still helps with the slab copies and barriers
    const int nrows_w = (EPI == EPI_SWIGLU) ? 2 * a.N : a.N;

    const char *W = reinterpret_cast<const char *>(a.W);
    const char *wrow[NT]; // byte pointers: this lane's row at its lane group's offset
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        int n = n0[t] + c;
        if (n > nrows_w - 1) n = nrows_w - 1; // ragged last tile: load a valid row, masked at the store
        wrow[t] = W + ((size_t)n * K + g * E) * sizeof(T);
    }
    const T *act = reinterpret_cast<const T *>(a.act);
    // split-K (a.ksplit > 1): workgroup z multiplies K slabs [s_lo, s_hi) only and leaves raw partial tiles
    const int nslab_all = (K + WIDE_KS - 1) / WIDE_KS;
    const int s_lo = a.ksplit > 1 ? blockIdx.z * a.kslabs : 0;
    const int s_hi = a.ksplit > 1 ? min(s_lo + a.kslabs, nslab_all) : nslab_all;
    const int nslab = s_hi - s_lo;
    // the workgroup's slabs in rotated order (see gemm_cols_kernel: workgroups that walk K in step meet in the same memory
    // channels and activation lines); a request past the end repeats the last slab of the rotated order
    const int rot = k_rotation(nslab);
    auto slab_at = [&](int sl) { return s_lo + rotated(min(sl, nslab - 1), rot, nslab); };
    const int k_end = min(K, s_hi * WIDE_KS);

    // slab s -> LDS: this wave's DPW instructions; lane l brings row (l / 16) of its 4-row group, LDS unit l % 16
    typedef const void __attribute__((address_space(1))) *gptr;
    typedef void __attribute__((address_space(3))) *lptr;
    const int r4 = lane >> 4, q = lane & 15;
    auto slab_dma = [&](int sl, unsigned char *buf) {
        const int k0 = slab_at(sl) * WIDE_KS; // past the end: any valid slab (never multiplied)
#pragma unroll
        for (int i = 0; i < DPW; ++i) {
            const int grp = min(wave * DPW + i, GROUPS - 1); // a surplus instruction repeats the last group
            const int row = 4 * grp + r4;
            const int k = min(k0 + (q ^ (row & 15)) * EPU, a.ld_act - EPU);
            const T *src = act + (size_t)min(rt0 * 16 + row, a.R - 1) * a.ld_act + k;
            __builtin_amdgcn_global_load_lds((gptr)src, (lptr)(buf + grp * 1024), 16, 0, 0);
        }
        asm volatile("" ::: "memory");
    };
    auto w_load = [&](int sl, u32x4 (&w)[NT][KBS]) {
        const int k0 = slab_at(sl) * WIDE_KS; // past the end: the last slab again (a cache hit; never multiplied)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int kb = 0; kb < KBS; ++kb) {
                const int k = k0 + kb * 4 * E;
                w[t][kb] = ld16_global(wrow[t] + (size_t)min(k, K - (g + 1) * E) * sizeof(T)); // zeroed past K when it is used
            }
        asm volatile("" ::: "memory");
    };

    // two accumulator sets per output tile (alternate k-blocks) so that
    // consecutive MFMAs never wait on each other
    f32x4 acc[2][RT][NT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[h][r][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Activation slabs are requested two steps ahead (three LDS buffers), and so are the weight slabs (three
    // register sets; deeper weight rings were measured and are slower).  A step issues [slab sl+2 -> LDS,
    // weights sl+2 -> registers]; buffers and register sets are compile-time choices, so the loop below is
    // unrolled over three steps and the last one or two steps of a slab count that is not a multiple of
    // three are written out after it (no idle step: the projections with K split four ways have 8 steps).
    u32x4 wring[3][NT][KBS];
    slab_dma(0, slab0);
    w_load(0, wring[0]);
    slab_dma(1, slab1);
    w_load(1, wring[1]);
    auto step = [&](int sl, const unsigned char *cur, unsigned char *fill, u32x4 (&wcur)[NT][KBS], u32x4 (&wfill)[NT][KBS]) {
        // this wave's part of slab sl and its weight slab sl have landed: the only younger loads are
        // those of the previous step (slab sl+1, weights sl+1)
        wait_vmcnt_at_most<DPW + WN>();
        wide_barrier(); // everybody's part has landed, and everybody is done reading `fill` (slab sl - 1)
        slab_dma(sl + 2, fill);
        w_load(sl + 2, wfill);
        const unsigned char *base = cur + (size_t)c * WIDE_SLAB_BYTES;
        // the LDS reads of k-block kb+1 are issued before the MFMAs of k-block kb (the scheduling
        // barriers keep the compiler from sinking them next to their uses, which serialises every
        // MFMA behind an LDS round trip)
        auto read_av = [&](int kb, Act<T> (&av)[RT]) {
#pragma unroll
            for (int r = 0; r < RT; ++r) av[r].p[0] = *reinterpret_cast<const u32x4 *>(base + (size_t)r * 16 * WIDE_SLAB_BYTES + (((kb * 4 + g) ^ c) * 16));
            __builtin_amdgcn_sched_barrier(0);
        };
        Act<T> av[2][RT];
        read_av(0, av[0]);
#pragma unroll
        for (int kb = 0; kb < KBS; ++kb) {
            if (kb + 1 < KBS) read_av(kb + 1, av[(kb + 1) & 1]);
            const bool in_k = slab_at(sl) * WIDE_KS + kb * KB + g * E < k_end;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const u32x4 wm = in_k ? wcur[t][kb] : zero16();
#pragma unroll
                for (int r = 0; r < RT; ++r) mma_split(acc[0][r][t], acc[1][r][t], wm, av[kb & 1][r], kb);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int s0 = 0;
    for (; s0 + 3 <= nslab; s0 += 3) {
        step(s0, slab0, slab2, wring[0], wring[2]);
        step(s0 + 1, slab1, slab0, wring[1], wring[0]);
        step(s0 + 2, slab2, slab1, wring[2], wring[1]);
    }
    if (s0 < nslab) step(s0, slab0, slab2, wring[0], wring[2]);
    if (s0 + 1 < nslab) step(s0 + 1, slab1, slab0, wring[1], wring[0]);
    wait_vmcnt_at_most<0>(); // nothing may still be landing in LDS when the workgroup ends
    move_lengths<EPI>(a);
    if (!tile_live) return;
    const int row_tiles = (a.R + 15) / 16;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        float out[NT][4];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) out[t][v] = acc[0][r][t][v] + acc[1][r][t][v];
        if (a.ksplit > 1) {
            if (EPI == EPI_RESID && a.splitk_rows) { // plain rows [split][R][N]: the launch that follows works row by row
                const int row = (rt0 + r) * 16 + c;
                if (row < a.R)
                    *reinterpret_cast<float4 *>(a.splitk_ws + ((size_t)blockIdx.z * a.R + row) * a.N + n0[0] + 4 * g) =
                        make_float4(out[0][0], out[0][1], out[0][2], out[0][3]);
            } else if (rt0 + r < row_tiles) {
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) a.splitk_ws[splitk_index(blockIdx.z, ntiles, tile, row_tiles, rt0 + r, NT, t, v, lane)] = out[t][v];
            }
        } else {
            apply_epilogue<T, EPI>(a, out, n0, rt0 + r);
        }
    }
}

// Second pass of a split-K launch: one wave per (wave tile, row tile) sums the splits' partial tiles in
// split order and runs the epilogue.  grid (wave tiles, row tiles).
template <int EPI>
__global__ __launch_bounds__(64) void gemm_splitk_finish_kernel(GemmArgs a) {
    constexpr int NT = (EPI == EPI_SWIGLU || EPI == EPI_QKV) ? 2 : 1;
    const int lane = threadIdx.x, tile = blockIdx.x, rt = blockIdx.y, row_tiles = gridDim.y;
    int n0[NT];
    const int ntiles = wide_tile_cols<EPI>(a, tile, n0);
    float out[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float s = 0.f;
            for (int z = 0; z < a.ksplit; ++z) s += a.splitk_ws[splitk_index(z, ntiles, tile, row_tiles, rt, NT, t, v, lane)];
            out[t][v] = s;
        }
    apply_epilogue<float, EPI>(a, out, n0, rt);
}

// Matrices with few column tiles would leave most of the chip idle (one workgroup per compute unit fits:
// 64 workgroups for a 4096-column projection).  K is then split over up to 4 workgroups whose partial
// tiles a second small launch sums in a fixed order; the split count is the largest that still fits the
// chip in one round, so the extra traffic (partials written and read once) stays a fraction of the weights.
// A residual projection (whole 16-column tiles, dense output rows) leaves its partials as plain rows, and the
// second launch is the RMSNorm kernel with the sum over the splits in front: it completes h and, when the caller
// named the norm that follows, writes that too (returns true then).
template <int EPI, int NW, int RT> static int launch_wide(const GemmArgs &a0, int tiles, int row_tiles, hipStream_t st) {
    constexpr int NT = (EPI == EPI_SWIGLU || EPI == EPI_QKV) ? 2 : 1;
    constexpr int WIDE_KS = WIDE_SLAB_BYTES / (int)sizeof(float);
    GemmArgs a = a0;
    const int gx = (tiles + NW - 1) / NW, gy = (row_tiles + RT - 1) / RT;
    const int nslab = (a.K + WIDE_KS - 1) / WIDE_KS;
    int ks = std::min(std::min(256 / std::max(gx * gy, 1), 4), nslab);
    a.ksplit = 1;
    a.kslabs = nslab;
    if (ks > 1 && a.splitk_ws) {
        const int per = (nslab + ks - 1) / ks;
        ks = (nslab + per - 1) / per; // no empty split
        const size_t need = sizeof(float) * (size_t)ks * tiles * row_tiles * NT * 256;
        if (ks > 1 && need <= a.splitk_ws_bytes) {
            a.ksplit = ks;
            a.kslabs = per;
        }
    }
    a.splitk_rows = EPI == EPI_RESID && a.ksplit > 1 && a.ksplit <= 4 && a.N % 16 == 0 && a.ldo == a.N && a.out == a.resid;
    hipLaunchKernelGGL((gemm_wide_kernel<EPI, NW, RT>), dim3(gx, gy, a.ksplit), dim3(NW * 64), 0, st, a);
    if (a.splitk_rows) {
        launch_splitk_resid_norm(0, a.out, a.splitk_ws, a.ksplit, a.norm_gain, a.R, a.N, a.norm_eps,
                                 a.norm_act, a.norm_act_plane, a.norm_ld, st);
        return a.norm_gain != nullptr ? 1 : 0;
    }
    if (a.ksplit > 1) hipLaunchKernelGGL((gemm_splitk_finish_kernel<EPI>), dim3(tiles, row_tiles), dim3(64), 0, st, a);
    return 0;
}

// More than 16 rows, bf16, int8 and int4 matrices.  A workgroup multiplies BM = 16 * RTW * WR rows (two planes of activations) with 16 * CT columns;
// both operands of a stage (KBS k-blocks of 32 K entries) come by load-to-LDS instructions, whole 128- or 256-byte pieces of a
// row, and are read back as operands (16-byte units of a row at position unit xor row: no bank conflicts).  The wavefronts split
// the rows WR ways, the columns WC ways and the k-blocks of a stage WK ways (their sums meet in LDS at the end), each keeps
// RTW x CTW tiles in registers: with one column tile per wavefront, as in the kernel below, every 10 - 20 MFMAs cost 10 KB of LDS reads.
//   What bounds it: up to about 100 rows the loads.  The weights have one trip through memory, the activations come from the L2 at 116 GB/s
// per compute unit (80 rows of K 4096: 14 us) and both share one path, so loads alone take their sum: 80 rows x 96 columns 35 us a launch
// of 22016 columns, the kernel 48.  They got there by
//   - a ring of ABUF stages of activations and WBUF of the matrix, the matrix's one stage deeper where LDS does not hold three of both (loads
//     alone, one | two stages ahead: 45 | 37 us), asked for in that order, so that the counted wait leaves the younger ones in flight;
//   - 256 bytes of a row at a time where LDS allows (128: 40 us) and the non-temporal bit on the matrix's (37.4 -> 34.7; launch_tile_as says when);
//   - a start in K that depends on the XCD: its workgroups walk K together and find each other's activations in their L2, the eight XCDs
//     ask different memory channels (no rotation 38 us, every workgroup its own 35.4; 256 rows, where the activations fill an L2: 71, 99, 67);
//   - row blocks of the same columns on one XCD, next to one another in time (tile_place): weights of two blocks from memory once (52 -> 37 us).
// With 128 rows and more to a block a launch is bound by the power of the card: 256 rows of 4096 x 22016 take 100 us, the same launch on zeros 79,
// its loads alone 76, its MFMAs and LDS reads alone 64.  (MFMAs of 32 x 32: 113 us; requests between the MFMAs: 100; the two wavefronts
// of a SIMD half a step apart: 107.)  More wavefronts of smaller tiles pay where a wavefront's MFMAs, requests and LDS reads stand behind
// one another (4 -> 8 waves, 128 x 64: 34 -> 29 us; 4 -> 12, 80 x 96: 52 -> 48), not where they read the LDS twice as often.
//   Measured (7B shape, us, before this form of it -> now; R rows, QKV and O / down with their second launches): gate/up 256 rows 109 -> 100,
// 192 112 -> 74, 72 53.6 -> 48, 40 47.8 -> 34, 24 47 -> 31; QKV 256 rows 68 -> 58, 192 68 -> 50, 40 28 -> 27; down 192 rows 57 -> 43.
//   A wavefront's load instructions are its share and no more (surplus ones that repeat the last: 3 - 6 % of every launch).
//   Quantised matrices are staged as they are and converted where they are read as operands, eight entries a lane and k-block: the loads shrink
// by what the entries do, conversions take their place.  int8: the row's scale on the finished sums.  int4: a stage is one scale
// group; its sums start at zero, a column tile at a time, and are added times the group's scales, which come with the stage.  Against the
// column-per-wavefront kernel, 2 layers of 7B shape, us: int8 24 rows 204 -> 165, 72 314 -> 234, 128 503 -> 324, 256 857 -> 505; int4 198 -> 181, 327 ->
// 263, 539 -> 334, 922 -> 525 (bf16: 212, 275, 328, 485).
template <int QB_, int RTW_, int CTW_, int WR_, int WC_, int WK_, int KBS_, int ABUF_, int WBUF_> struct TileCfg {
    static constexpr int QB = QB_; // bits of a quantised matrix, 0: bf16
    static constexpr int RTW = RTW_, CTW = CTW_, WR = WR_, WC = WC_, WK = WK_, KBS = KBS_, ABUF = ABUF_, WBUF = WBUF_;
    static constexpr int NW = WR * WC * WK;         // wavefronts
    static constexpr int BM = 16 * RTW * WR;        // rows
    static constexpr int CT = CTW * WC;             // 16-column tiles
    static constexpr int ROWB = 64 * KBS, WROWB = QB ? ROWB * QB / 16 : ROWB; // bytes of a row in a stage (KBS k-blocks of 32 entries): activations, matrix
    static constexpr int UPR = ROWB / 16, WUPR = WROWB / 16;                   // ... in 16-byte units
    static constexpr int RPI = 64 / UPR, WRPI = 64 / WUPR;                     // rows per load instruction
    static constexpr int SCALES = QB == 4 ? (16 * CT + 63) / 64 : 0;           // int4: load instructions (of a word per lane) for the stage's scales
    static constexpr int ASTAGE = 2 * BM * ROWB, WBYTES = 16 * CT * WROWB, WSTAGE = WBYTES + 256 * SCALES; // a stage's two activation planes, its piece of the matrix
    // load instructions of a stage: activations, matrix (and scales), dealt out to the wavefronts in turn; most and fewest of a wavefront
    static constexpr int AG = 2 * BM / RPI, WG = 16 * CT / WRPI, WS = WG + SCALES;
    static constexpr int AL = (AG + NW - 1) / NW, AMIN = AG / NW, WL = (WS + NW - 1) / NW, WMIN = WS / NW;
    // 16-byte unit u of row r of the matrix lies at position u xor (r mod 8 or 16), with four units a row u xor (r / 2 mod 4): sixteen rows'
    // units are in different banks
    static __device__ __forceinline__ int swizzle(int row) { return WUPR == 4 ? (row >> 1) & 3 : row & (WUPR - 1); }
    static_assert(QB != 4 || KBS == 4, "an int4 stage is a scale group");
    static_assert(WUPR >= 4, "");
    static constexpr int LDS = ABUF * ASTAGE + WBUF * WSTAGE;
    static_assert(LDS <= 160 * 1024 && WBUF >= ABUF && ABUF >= 2 && WBUF <= 3, "");
};

__device__ __forceinline__ void stage_barrier() { // ... which no LDS access may cross
    asm volatile("" ::: "memory");
    wide_barrier();
    asm volatile("" ::: "memory");
}

// The workgroup's place: the row blocks of a column share lie on one XCD (workgroups go round the eight of them), next to one another in time,
// so that the second reads the weights of the first from their L2.
struct TilePlace {
    int x, y, id; // column share, row block, number in launch order (of a split)
};
__device__ __forceinline__ TilePlace tile_place() {
    if (gridDim.y == 1) return TilePlace{(int)blockIdx.x, 0, (int)blockIdx.x}; // (no divisions in front of the first load)
    const int gx = gridDim.x, gy = gridDim.y, id = blockIdx.x + gx * blockIdx.y, whole = (gx & ~7) * gy;
    if (id >= whole) {
        const int rest = id - whole, w = gx & 7;
        return TilePlace{(gx & ~7) + rest % w, rest / w, id};
    }
    const int slot = id >> 3;
    return TilePlace{slot / gy * 8 + (id & 7), slot % gy, id};
}

template <int EPI, class C>
__global__ __launch_bounds__(C::NW * 64) void gemm_tile_kernel(GemmArgs a) {
    typedef bf16_t T;
    constexpr int NT = (EPI == EPI_SWIGLU || EPI == EPI_QKV) ? 2 : 1;
    constexpr int RTW = C::RTW, CTW = C::CTW, WK = C::WK, KBS = C::KBS, ABUF = C::ABUF, WBUF = C::WBUF, NW = C::NW;
    constexpr int QB = C::QB;
    static_assert(CTW % NT == 0 && KBS % WK == 0, "");
    __shared__ __align__(16) unsigned char lds[C::LDS];
    const uint32_t lds0 = lds_address(lds);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int wk = wave / (NW / WK), wc = wave % C::WC, wr = wave % (NW / WK) / C::WC;
    const int K = a.K;
    const TilePlace place = tile_place();
    const int row0 = place.y * C::BM;
    // first column of output tile `ct` of the workgroup (fused epilogues: tiles 2p and 2p + 1 are the two halves of pair p)
    const int npairs = EPI == EPI_QKV ? 3 * a.H * (a.hd / 32) : (a.N + 15) / 16;
    const int nrows_w = EPI == EPI_SWIGLU ? 2 * a.N : a.N;
    auto tile_col = [&](int ct) {
        const int p = min(place.x * (C::CT / NT) + ct / NT, npairs - 1), half = ct % NT;
        if constexpr (EPI == EPI_QKV) {
            const int per_head = a.hd / 32, hh = p / per_head;
            return hh * a.hd + (p % per_head) * 16 + half * (a.hd / 2);
        } else if constexpr (EPI == EPI_SWIGLU) {
            return p * 16 + half * a.N;
        } else {
            return p * 16;
        }
    };
    const int nst_all = (K + 32 * KBS - 1) / (32 * KBS);
    const int s_lo = a.ksplit > 1 ? blockIdx.z * a.kslabs : 0;
    const int nst = (a.ksplit > 1 ? min(s_lo + a.kslabs, nst_all) : nst_all) - s_lo;
    const int rot = (place.id & 7) * nst / 8; // (see TileCfg)
    auto stage_at = [&](int s) { return s_lo + rotated(s, rot, nst); };

    // this wave's load instructions of a stage: of the activations wave + i * NW, of the matrix (int4: the scales behind it) wwave + i * NW; lane l
    // brings unit (l % UPR) xor row of row l / UPR
    const int wwave = wave < C::AG % NW ? wave - C::AG % NW + NW : wave - C::AG % NW; // the first ones go to those with fewer of the activations
    const int na = C::AMIN + (wave < C::AG % NW), nw = C::WMIN + (wwave < C::WS % NW);
    const size_t row_bytes = QB ? (size_t)K * QB / 8 : (size_t)K * 2;
    const char *abase[C::AL], *wbase[C::WL];
    uint32_t aoff[C::AL], woff[C::WL];
    const int lr = lane / C::UPR, lu = lane % C::UPR, wlr = lane / C::WUPR, wlu = lane % C::WUPR;
#pragma unroll
    for (int i = 0; i < C::AL; ++i) {
        const int r0 = min(wave + i * NW, C::AG - 1) * C::RPI, row = r0 + lr, pl = r0 / C::BM, r = row - pl * C::BM;
        abase[i] = reinterpret_cast<const char *>(reinterpret_cast<const T *>(a.act) + pl * a.act_plane + (size_t)min(row0, a.R - 1) * a.ld_act);
        aoff[i] = (uint32_t)(min(row0 + r, a.R - 1) - min(row0, a.R - 1)) * (uint32_t)a.ld_act * 2u + (uint32_t)(lu ^ (row & (C::UPR - 1))) * 16u;
    }
#pragma unroll
    for (int i = 0; i < C::WL; ++i) {
        const int grp = wwave + i * NW;
        if (QB == 4 && grp >= C::WG) {
            const int w = min((grp - C::WG) * 64 + lane, 16 * C::CT - 1);
            wbase[i] = reinterpret_cast<const char *>(a.wscale);
            woff[i] = (uint32_t)min(tile_col(w / 16) + (w & 15), nrows_w - 1) * 4u;
        } else {
            const int row = min(grp, C::WG - 1) * C::WRPI, n0 = tile_col(row / 16), n = min(n0 + (row & 15) + wlr, nrows_w - 1);
            wbase[i] = reinterpret_cast<const char *>(a.W) + (size_t)n0 * row_bytes;
            woff[i] = (uint32_t)(n - n0) * (uint32_t)row_bytes + (uint32_t)(wlu ^ C::swizzle(row + wlr)) * 16u;
        }
    }
    // (Never with int4.  A constant there: the rows and units that only a ragged end needs took the registers of two addresses in the 80 x 192 tile of QKV, and the
    // wait behind each of their spills emptied the ring: three layers of 7B | 13B shape,
    // 72 rows, us: 398.0 -> 386.1 | 554.5 -> 531.8, and 18 rows, which spilled nothing, 272.0 -> 262.9 | 357.4 -> 345.9.)
    const bool ragged = QB != 4 && K % (32 * KBS) != 0;
    auto issue_act = [&](int s, int buf) {
        const int st = stage_at(s);
        const uint32_t to = lds0 + buf * C::ASTAGE + wave * 1024;
        const size_t kb = (size_t)st * C::ROWB;
#pragma unroll
        for (int i = 0; i < C::AL; ++i)
            if (i < C::AMIN || i < na) {
                // past a ragged end: units past K repeat the row's last one (their weights are zeroed when used)
                const int row = (wave + i * NW) * C::RPI + lr;
                const uint32_t over = ragged && st == nst_all - 1 ? (uint32_t)max(st * C::ROWB + (lu ^ (row & (C::UPR - 1))) * 16 - (2 * K - 16), 0) : 0u;
                dma16(abase[i] + kb, aoff[i] - over, to + i * NW * 1024);
            }
    };
    auto issue_w = [&](int s, int buf) {
        const int st = stage_at(s);
        const uint32_t to = lds0 + ABUF * C::ASTAGE + buf * C::WSTAGE;
        const size_t kb = (size_t)st * C::WROWB;
#pragma unroll
        for (int i = 0; i < C::WL; ++i)
            if (i < C::WMIN || i < nw) {
                const int grp = wwave + i * NW;
                if (QB == 4 && grp >= C::WG) {
                    dma4(wbase[i] + (size_t)st * nrows_w * 4, woff[i], to + C::WBYTES + (grp - C::WG) * 256);
                } else {
                    const uint32_t over = ragged && st == nst_all - 1 ? (uint32_t)max(st * C::WROWB + (wlu ^ C::swizzle(grp * C::WRPI + wlr)) * 16 - ((int)row_bytes - 16), 0) : 0u;
                    if (a.stream) dma16<true>(wbase[i] + kb, woff[i] - over, to + grp * 1024);
                    else dma16(wbase[i] + kb, woff[i] - over, to + grp * 1024);
                }
            }
    };
    f32x4 acc[RTW][CTW];
#pragma unroll
    for (int r = 0; r < RTW; ++r)
#pragma unroll
        for (int t = 0; t < CTW; ++t) acc[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // waits for stage s: younger are only the stages requested ahead of it
    auto wait_stage = [&](int s) {
        const int wa = min(WBUF - 2, nst - 1 - s), aa = min(ABUF - 2, nst - 1 - s);
        constexpr int AF = ABUF - 2, WF = WBUF - 2;
        if (AF && aa > 0) wait_vmcnt<AF * C::AMIN + WF * C::WMIN, AF * C::AL + WF * C::WL>(AF * na + WF * nw);
        else if (WF && wa > 0) wait_vmcnt<WF * C::WMIN, WF * C::WL>(WF * nw);
        else wait_vmcnt_at_most<0>();
    };
    // Which K entries lane (c, g) supplies to k-block kb of a stage is free as long as both operands agree.  bf16: unit 4 kb + g of a row.  int8:
    // half kb % 2 of unit 4 (kb / 2) + g of the matrix, 8 entries, unit 8 (kb / 2) + 2g + kb % 2 of the activations.  int4: dword kb of
    // unit g, 8 entries, unit 4g + kb.
    auto act_unit = [&](int kb) { return QB == 4 ? 4 * g + kb : QB == 8 ? 8 * (kb >> 1) + 2 * g + (kb & 1) : 4 * kb + g; };
    auto read_act = [&](int ab, int kb, u32x4 (&b)[RTW][2]) {
        const int un = (act_unit(kb) ^ (c & (C::UPR - 1))) * 16; // (the xor only touches the low bits of the row, which is c's for every tile)
        const unsigned char *ap = lds + ab * C::ASTAGE;
#pragma unroll
        for (int r = 0; r < RTW; ++r)
#pragma unroll
            for (int pl = 0; pl < 2; ++pl) b[r][pl] = *reinterpret_cast<const u32x4 *>(ap + (pl * C::BM + (wr * RTW + r) * 16 + c) * C::ROWB + un);
    };
    auto mma1 = [&](f32x4 s, u32x4 w, u32x4 b) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, b), s, 0, 0, 0); };
    auto compute = [&](int s, int ab, int wb) {
        constexpr int KK = KBS / WK; // k-blocks of this wavefront
        const unsigned char *wp = lds + ABUF * C::ASTAGE + wb * C::WSTAGE;
        if constexpr (QB == 4) {
            // the stage is one scale group: its sums, a column tile at a time, times the scales of the lane's four columns
            typedef uint32_t dwords __attribute__((ext_vector_type(KK)));
            u32x4 b[KK][RTW][2];
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) read_act(ab, wk * KK + kk, b[kk]);
#pragma unroll
            for (int t = 0; t < CTW; ++t) {
                const int tile = wc * CTW + t;
                const dwords q = *reinterpret_cast<const dwords *>(wp + (tile * 16 + c) * C::WROWB + (g ^ C::swizzle(c)) * 16 + 4 * wk * KK);
                const f32x4 sc = *reinterpret_cast<const f32x4 *>(wp + C::WBYTES + (tile * 16 + 4 * g) * 4);
                f32x4 part[RTW];
#pragma unroll
                for (int r = 0; r < RTW; ++r) part[r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) {
                    const u32x4 w = w4_to_bf16x8_sixteenths(q[kk]);
#pragma unroll
                    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                        for (int r = 0; r < RTW; ++r) part[r] = mma1(part[r], w, b[kk][r][pl]);
                }
#pragma unroll
                for (int r = 0; r < RTW; ++r)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[r][t][v] += sc[v] * part[r][v];
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const int kb = wk * KK + kk;
                u32x4 w[CTW], b[RTW][2];
                uint2 q[CTW];
#pragma unroll
                for (int t = 0; t < CTW; ++t) {
                    const unsigned char *row = wp + ((wc * CTW + t) * 16 + c) * C::WROWB;
                    if constexpr (QB == 8) q[t] = *reinterpret_cast<const uint2 *>(row + ((4 * (kb >> 1) + g) ^ C::swizzle(c)) * 16 + 8 * (kb & 1));
                    else w[t] = *reinterpret_cast<const u32x4 *>(row + ((4 * kb + g) ^ C::swizzle(c)) * 16);
                }
                read_act(ab, kb, b);
                if (ragged && stage_at(s) == nst_all - 1 && (nst_all - 1) * 32 * KBS + act_unit(kb) * 8 >= K) {
#pragma unroll
                    for (int t = 0; t < CTW; ++t) {
                        if constexpr (QB == 8) q[t] = make_uint2(0u, 0u);
                        else w[t] = zero16();
                    }
                }
                if constexpr (QB == 8) {
#pragma unroll
                    for (int t = 0; t < CTW; ++t) w[t] = w8_to_bf16x8(q[t].x, q[t].y);
                }
#pragma unroll
                for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                    for (int r = 0; r < RTW; ++r)
#pragma unroll
                        for (int t = 0; t < CTW; ++t) acc[r][t] = mma1(acc[r][t], w[t], b[r][pl]);
            }
        }
    };
#pragma unroll
    for (int s = 0; s < WBUF - 1; ++s) {
        if (s < ABUF - 1 && s < nst) issue_act(s, s);
        if (s < nst) issue_w(s, s);
    }
    for (int s = 0, ab = 0, wb = 0; s < nst; ++s) {
        wait_stage(s);
        stage_barrier(); // everybody's part of the stage has landed, and everybody is done reading the ones that are filled next
        if (s + ABUF - 1 < nst) issue_act(s + ABUF - 1, ab == 0 ? ABUF - 1 : ab - 1);
        if (s + WBUF - 1 < nst) issue_w(s + WBUF - 1, wb == 0 ? WBUF - 1 : wb - 1);
        compute(s, ab, wb);
        ab = ab == ABUF - 1 ? 0 : ab + 1;
        wb = wb == WBUF - 1 ? 0 : wb + 1;
    }

    auto finish = [&](float (&out)[NT][4], int r, int p) { // row tile r and column tile (pair) p of the workgroup
        if constexpr (QB == 4) { // (the entries were sixteenths)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) out[t][v] *= 16.0f;
        }
        const int ct = p * NT;
        if (place.x * (C::CT / NT) + p >= npairs) return;
        int n0[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) n0[t] = tile_col(ct + t);
        const int m = row0 + r * 16 + c;
        if constexpr (QB == 8) { // (linear: also right for partial sums)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) out[t][v] *= a.wscale[min(n0[t] + 4 * g + v, nrows_w - 1)];
        }
        if ((EPI == EPI_RESID || EPI == EPI_QKV) && a.ksplit > 1) { // plain rows [split][R][N]: the launch that follows works row by row
            if (m < a.R) {
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    *reinterpret_cast<float4 *>(a.splitk_ws + ((size_t)blockIdx.z * a.R + m) * a.N + n0[t] + 4 * g) = make_float4(out[t][0], out[t][1], out[t][2], out[t][3]);
            }
        } else {
            apply_epilogue<T, EPI>(a, out, n0, row0 / 16 + r);
        }
    };
    if constexpr (WK == 1) {
#pragma unroll
        for (int r = 0; r < RTW; ++r)
#pragma unroll
            for (int p = 0; p < CTW / NT; ++p) {
                float out[NT][4];
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) out[t][v] = acc[r][p * NT + t][v];
                finish(out, wr * RTW + r, wc * (CTW / NT) + p);
            }
    } else {
        // the K shares of a tile are summed in order through LDS, a row tile at a time in alternating buffers
        static_assert(2 * NW * CTW * 1024 <= C::LDS, "");
#pragma unroll
        for (int r = 0; r < RTW; ++r) {
            float *red = reinterpret_cast<float *>(lds + (r & 1) * (NW * CTW * 1024));
            if (r == 0) stage_barrier(); // nobody reads the stages any more
#pragma unroll
            for (int t = 0; t < CTW; ++t) *reinterpret_cast<f32x4 *>(red + ((size_t)(wave * CTW + t) * 64 + lane) * 4) = acc[r][t];
            stage_barrier();
#pragma unroll
            for (int p = 0; p < CTW / NT; ++p)
                if (p % WK == wk) {
                    float out[NT][4];
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int k2 = 0; k2 < WK; ++k2)
                            sum += *reinterpret_cast<const f32x4 *>(red + ((size_t)((wave % (NW / WK) + k2 * (NW / WK)) * CTW + p * NT + t) * 64 + lane) * 4);
#pragma unroll
                        for (int v = 0; v < 4; ++v) out[t][v] = sum[v];
                    }
                    finish(out, wr * RTW + r, wc * (CTW / NT) + p);
                }
        }
    }
    move_lengths<EPI>(a);
}

// Second launch of a split QKV projection: four column pairs of a row per thread, the splits added in order.  A workgroup takes 16
// rows x 16 quads, neighbouring lanes neighbouring rows: a value column of the cache has its positions side by side, two bytes
// each (a row per workgroup wrote every one of them to a line of its own: 72 rows 10.6 -> 8.1 us, 256 rows 19 -> 15).
// grid (rows / 16, quads / 16)
__global__ __launch_bounds__(256) void qkv_finish_kernel(GemmArgs a) {
    const int m = blockIdx.x * 16 + (threadIdx.x & 15), half = a.hd / 2, quads = half / 4; // quads of pairs per head
    const int i = blockIdx.y * 16 + (threadIdx.x >> 4), hh = i / quads;
    if (hh >= 3 * a.H || m >= a.R) return;
    const int j0 = 4 * (i - hh * quads);
    const float *p = a.splitk_ws + (size_t)m * a.N + hh * a.hd + j0;
    float4 lo[4], hi[4];
#pragma unroll
    for (int z = 0; z < 4; ++z) { // (all requested before the first is used; at most four splits)
        const size_t at = (size_t)min(z, a.ksplit - 1) * a.R * a.N;
        lo[z] = *reinterpret_cast<const float4 *>(p + at);
        hi[z] = *reinterpret_cast<const float4 *>(p + at + half);
    }
    float x0[4] = {lo[0].x, lo[0].y, lo[0].z, lo[0].w}, x1[4] = {hi[0].x, hi[0].y, hi[0].z, hi[0].w};
#pragma unroll
    for (int z = 1; z < 4; ++z)
        if (z < a.ksplit) {
            x0[0] += lo[z].x; x0[1] += lo[z].y; x0[2] += lo[z].z; x0[3] += lo[z].w;
            x1[0] += hi[z].x; x1[1] += hi[z].y; x1[2] += hi[z].z; x1[3] += hi[z].w;
        }
    epilogue_cols<bf16_t, EPI_QKV, 4>(a, m, hh * a.hd + j0, x0, x1);
}

// Which tile and which split of K: the least of  rounds * (1.1 us + K share * (A us/MB * activations + W us/MB * weights)) + 3 ns a workgroup
// over the shapes there are; A and W were fitted to 40 launches of 2048- to 5120-wide models at 17 to 256 rows (they are within 8 % of
// what those take on average, and the choice within 2 % of the best one; 5 - 7 % for QKV of up to 48 rows, where 192 columns are taken and
// 96 would be 1.2 us faster).  A: 9 in stages of 128 bytes a row, 13.5 in stages of 256 with three of them in LDS, 15 with two.  W: 31 in
// stages of 256 bytes, 26 in blocks of 128 rows with up to 96 columns, 29 for 128 columns, 32.5 for 192, 34.5 with several row blocks.  A
// split adds its partial rows, written and read once (8 MB/us), 0.16 us of the second launch and for QKV that launch (4.5 us; a residual
// projection's is the RMSNorm that follows anyway).  Quantised matrices (bits < 16), where conversions and MFMAs weigh more than the bytes, take
// 2 ns (int4: 3) and 0.81 ps (0.875) an output for every K entry: seven tiles of a 4096 x 22016 matrix within 10 %.
struct TileChoice {
    int rows, cols, ksplit;
    double us;
};
//   Two tiles are priced otherwise than they are built: gate and up in 48 rows x 128 columns with two stages of activations at 13.5, a head of one round in 48 x 128
// with stages of 256 bytes at 9 and 29.  With 15, and with 15 and 31, they would be taken at the same sizes (10.8 ns for every entry of K against
// 14.2 in 192 columns and two rounds of 8.5 in 96; against two rounds of 6.6 in 64).
//   Many rows of a short K (bf16) have an older form of the sum, 16 us/MB of activations and 40 (several row blocks: 34) of the matrix and no start:
// launches of one to sixteen stages are bound by their ends, and the terms above, fitted to long ones, chose blocks of 128 rows and splits there.  1024 rows, a
// layer of d_model 128 | 256 | 512, us: 39.3 -> 36.9 | 57.4 -> 52.1 | 71.2 -> 69.8.
static TileChoice tile_cost(int epi, int bits, int bm, int cols, int columns, int R, int K, int ksplit, double launch_us, bool short_k) {
    const int gy = (R + bm - 1) / bm, gx = (columns + cols - 1) / cols, wgs = gx * gy * ksplit;
    const int rounds = (wgs + 255) / 256;
    const double second = ksplit > 1 ? launch_us + 8.0 * ksplit * R * columns / 8e6 : 0.0;
    if (short_k && bits == 16) return TileChoice{bm, cols, ksplit, rounds * (double)((K + ksplit - 1) / ksplit) * (bm * 4 * 16e-6 + cols * 2 * (gy > 1 ? 34e-6 : 40e-6)) + second};
    const bool fused = epi == EPI_SWIGLU || epi == EPI_QKV;
    const bool long_stage = cols <= 96 ? bm <= 96 : fused && cols == 128 && bm <= 48; // 256 bytes of a row
    const double act = !long_stage ? 9e-6 : bm <= 48 ? 13.5e-6 : 15e-6;
    const double mat = long_stage ? 31e-6 : cols <= 96 ? 26e-6 : cols == 128 ? 29e-6 : gy > 1 ? 34.5e-6 : 32.5e-6;
    const double per = bits == 16 ? bm * 4 * act + cols * 2 * mat : bits == 8 ? 2.0e-3 + 8.1e-7 * bm * cols : 3.0e-3 + 8.75e-7 * bm * cols;
    return TileChoice{bm, cols, ksplit, rounds * (1.1 + (double)((K + ksplit - 1) / ksplit) * per) + 0.003 * wgs + second + (ksplit > 1 ? 0.16 * ksplit : 0.0)};
}

template <int EPI, class C> static int launch_tile_as(const GemmArgs &a0, int columns, int ksplit, hipStream_t st) {
    GemmArgs a = a0;
    const int nst = (a.K + 32 * C::KBS - 1) / (32 * C::KBS);
    a.kslabs = (nst + ksplit - 1) / ksplit;
    a.ksplit = (nst + a.kslabs - 1) / a.kslabs; // no empty split
    // The non-temporal bit on the matrix's requests: where the pass leaves nothing of the matrix in the memory-side cache (7B shape, gate/up
    // 24 | 40 | 72 rows 33.9 -> 30.9 | 36.2 -> 34.2 | 49.3 -> 47.8 us); what is still there comes later with the bit (one layer of 3B shape, 40
    // rows, 89.1 us with, 85.3 without; of 1B shape 68.4, 66.0).  Not for a residual projection, whose short splits lose by it (4096 x
    // 4096, 72 rows, 16.3 -> 17.5), nor where a stage takes half a line of a row (int4 gate/up of 72 rows 45.3 -> 47.0; int8 with whole lines, 2 layers of
    // 7B shape, 40 | 72 rows 208 -> 194 | 258 -> 245).
    a.stream = a0.stream && EPI != EPI_RESID && C::WROWB >= 128;
    hipLaunchKernelGGL((gemm_tile_kernel<EPI, C>), dim3((columns + 16 * C::CT - 1) / (16 * C::CT), (a.R + C::BM - 1) / C::BM, a.ksplit), dim3(C::NW * 64), 0, st, a);
    if (a.ksplit == 1) return 0;
    if constexpr (EPI == EPI_QKV) {
        hipLaunchKernelGGL(qkv_finish_kernel, dim3((a.R + 15) / 16, (3 * a.H * (a.hd / 8) + 15) / 16), dim3(256), 0, st, a);
        return 0;
    }
    launch_splitk_resid_norm(1, a.out, a.splitk_ws, a.ksplit, a.norm_gain, a.R, a.N, a.norm_eps, a.norm_act, a.norm_act_plane, a.norm_ld, st);
    return a.norm_gain != nullptr ? 1 : 0;
}

template <int EPI, int QB> static int launch_tile_as_chosen(const GemmArgs &a, int columns, const TileChoice &c, hipStream_t st) {
    auto go = [&](auto cfg) { return launch_tile_as<EPI, decltype(cfg)>(a, columns, c.ksplit, st); };
    constexpr bool FUSED = EPI == EPI_SWIGLU || EPI == EPI_QKV;
    const int tile = c.rows * 1000 + c.cols;
    if constexpr (QB != 0 && FUSED) {
        if constexpr (EPI == EPI_SWIGLU) {
            if (tile == 32128) return go(TileCfg<QB, 2, 2, 1, 4, 2, 4, 3, 3>{});
            if (tile == 48128) return go(TileCfg<QB, 3, 2, 1, 4, 2, 4, 3, 3>{});
            if (tile == 80128) return go(TileCfg<QB, 5, 2, 1, 4, 2, 4, 2, 3>{});
        }
        switch (tile) {
        case 32096: return go(TileCfg<QB, 2, 2, 1, 3, 4, 4, 3, 3>{});
        case 48096: return go(TileCfg<QB, 3, 2, 1, 3, 4, 4, 3, 3>{});
        case 80096: return go(TileCfg<QB, 5, 2, 1, 3, 4, 4, 3, 3>{});
        case 32192: return go(TileCfg<QB, 2, 2, 1, 6, 2, 4, 3, 3>{}); // (one round where 128 columns would make two)
        case 48192: return go(TileCfg<QB, 3, 2, 1, 6, 2, 4, 3, 3>{});
        case 80192: return go(TileCfg<QB, 5, 2, 1, 6, 2, 4, 2, 3>{});
        case 96096:
            if constexpr (QB == 4) return go(TileCfg<4, 3, 2, 2, 3, 2, 4, 2, 3>{});
            else return go(TileCfg<8, 3, 6, 2, 1, 4, 4, 2, 3>{});
        case 96192: return go(TileCfg<QB, 3, 6, 2, 2, 2, 4, 2, QB == 4 ? 3 : 2>{});
        case 128096: return go(TileCfg<QB, 4, 2, 2, 3, 2, 4, 2, QB == 4 ? 3 : 2>{});
        default: // 128 x 192
            if constexpr (QB == 4) return go(TileCfg<4, 4, 6, 2, 2, 2, 4, 2, 2>{});
            else return go(TileCfg<8, 4, 6, 2, 2, 2, 2, 2, 3>{});
        }
    } else if constexpr (QB != 0) {
        switch (tile) {
        case 32064: return go(TileCfg<QB, 2, 2, 1, 2, 4, 4, 3, 3>{});
        case 32128: // (heads: see below; int8, K 4096, 18 rows, 32000 | 40960 | 128256 columns 37.5 -> 36.7 | 59.4 -> 47.8 | 123.9 -> 105.8 us)
            if constexpr (EPI == EPI_STORE) return go(TileCfg<QB, 2, 2, 1, 4, 2, 4, 2, 2>{});
            else return go(TileCfg<QB, 2, 2, 1, 4, 2, 4, 3, 3>{});
        case 48064: return go(TileCfg<QB, 3, 2, 1, 2, 4, 4, 3, 3>{});
        case 48128: // (48 rows, one round of workgroups: 41.7 us with the deep rings, 45.0 with these; 40960 | 128256 columns 68.6 -> 55.3 | 149.8 -> 134.1)
            if constexpr (EPI == EPI_STORE) {
                if (columns > 128 * 256) return go(TileCfg<QB, 3, 2, 1, 4, 2, 4, 2, 2>{});
            }
            return go(TileCfg<QB, 3, 2, 1, 4, 2, 4, 3, 3>{});
        case 80064: return go(TileCfg<QB, 5, 2, 1, 2, 4, 4, 3, 3>{});
        case 80128: return go(TileCfg<QB, 5, 2, 1, 4, 2, 4, 2, 3>{});
        case 96128: return go(TileCfg<QB, 3, 4, 2, 2, 2, 4, 2, QB == 4 ? 3 : 2>{});
        default: // 128 x 128
            if constexpr (QB == 4) return go(TileCfg<4, 4, 4, 2, 2, 2, 4, 2, 2>{});
            else return go(TileCfg<8, 4, 4, 2, 2, 2, 2, 3, 3>{});
        }
    } else if constexpr (FUSED) {
        if constexpr (EPI == EPI_SWIGLU) {
            if (tile == 32128) return go(TileCfg<0, 2, 2, 1, 4, 2, 4, 3, 3>{});
            if (tile == 48128) return go(TileCfg<0, 3, 2, 1, 4, 2, 4, 2, 3>{});
            if (tile == 80128) return go(TileCfg<0, 5, 2, 1, 4, 2, 2, 3, 3>{});
        }
        switch (tile) {
        case 32064: return go(TileCfg<0, 2, 4, 1, 1, 4, 4, 3, 3>{});
        case 32096: return go(TileCfg<0, 2, 6, 1, 1, 4, 4, 3, 3>{});
        case 32192: return go(TileCfg<0, 2, 6, 1, 2, 2, 2, 3, 3>{});
        case 48064: return go(TileCfg<0, 3, 4, 1, 1, 4, 4, 3, 3>{});
        case 48096: return go(TileCfg<0, 3, 6, 1, 1, 4, 4, 3, 3>{});
        case 48192: return go(TileCfg<0, 3, 6, 1, 2, 2, 2, 3, 3>{});
        case 80064: return go(TileCfg<0, 5, 2, 1, 2, 4, 4, 2, 3>{});
        case 80096: return go(TileCfg<0, 5, 2, 1, 3, 4, 4, 2, 3>{});
        case 80192: return go(TileCfg<0, 5, 6, 1, 2, 2, 2, 3, 3>{});
        case 96096: return go(TileCfg<0, 3, 6, 2, 1, 4, 4, 2, 2>{});
        case 96192: return go(TileCfg<0, 3, 6, 2, 2, 2, 2, 3, 3>{});
        case 128096: return go(TileCfg<0, 2, 6, 4, 1, 2, 2, 3, 3>{});
        default: return go(TileCfg<0, 4, 6, 2, 2, 2, 2, 2, 3>{}); // 128 x 192
        }
    } else {
        switch (tile) {
        case 32064: return go(TileCfg<0, 2, 2, 1, 2, 4, 4, 3, 3>{});
        // Heads are several rounds of workgroups as a rule: rings of 64 to 80 KB, so that a compute unit holds two of them and one starts or ends while
        // the other streams.  K 4096, 18 rows, 32000 | 40960 | 128256 columns, one workgroup a unit (stages of 256 bytes a row, 128 KB) -> two:
        // 49.8 -> 49.6 | 83.1 -> 77.9 | 201.6 -> 185.3 us.  Of 48 rows only beyond one round: K 2048 31.2 -> 32.7 | 47.6 -> 42.7 | 115.3 -> 110.4,
        // K 4096 52.6 -> 54.8 | 86.3 -> 87.5 | 206.0 -> 200.6.
        case 32128:
            if constexpr (EPI == EPI_STORE) return go(TileCfg<0, 2, 2, 1, 4, 2, 2, 2, 3>{});
            else return go(TileCfg<0, 2, 2, 1, 4, 2, 2, 3, 3>{});
        case 48064: return go(TileCfg<0, 3, 2, 1, 2, 4, 4, 3, 3>{});
        case 48128:
            if constexpr (EPI == EPI_STORE) {
                if (columns > 128 * 256) return go(TileCfg<0, 3, 2, 1, 4, 2, 2, 2, 3>{});
                return go(TileCfg<0, 3, 2, 1, 4, 2, 4, 2, 3>{});
            } else {
                return go(TileCfg<0, 3, 2, 1, 4, 2, 2, 3, 3>{});
            }
        case 80064: return go(TileCfg<0, 5, 2, 1, 2, 4, 4, 2, 3>{});
        case 80128: return go(TileCfg<0, 5, 2, 1, 4, 2, 2, 3, 3>{});
        case 96064: return go(TileCfg<0, 3, 2, 2, 2, 2, 4, 2, 3>{});
        case 96128: return go(TileCfg<0, 3, 4, 2, 2, 2, 2, 3, 3>{});
        case 128064: return go(TileCfg<0, 2, 4, 4, 1, 2, 2, 3, 3>{});
        default: return go(TileCfg<0, 4, 4, 2, 2, 2, 2, 3, 3>{}); // 128 x 128
        }
    }
}

// tiles: 16-column tiles (pairs of them for the fused epilogues); ws_bytes: room for partial rows (0: K is not split)
static TileChoice choose_tile(int epi, int bits, int tiles, int R, int N, int K, size_t ws_bytes) {
    const bool fused = epi == EPI_SWIGLU || epi == EPI_QKV;
    const int columns = 16 * tiles * (fused ? 2 : 1);
    // rows per workgroup: 32, 48, 80 where that is all of them, else blocks of 128 - or of 80 or, beyond 160 rows, 96, where that pads less
    // (192 rows, us, blocks of 128 | 96: gate/up 93 | 75, QKV 59 | 50, O 25.8 | 22.7, down 51 | 43)
    const int p80 = (R + 79) / 80 * 80, p96 = (R + 95) / 96 * 96, p128 = (R + 127) / 128 * 128;
    const int bm0 = R <= 32 ? 32 : R <= 48 ? 48 : (R > 160 && p96 * 1.1 < std::min(p80, p128)) ? 96 : (R <= 80 || p80 * 1.1 < p128) ? 80 : 128;
    // Many rows of a short K: few such blocks leave most of the chip idle and splitting K cannot fill it (a share of less than 256 entries
    // is over before the ring is full, and the partial rows come on top), so the cost chooses the block as well.  1024 rows, a pass of
    // 2 layers, us: d_model 128 133 -> 81, 256 161 -> 115, 512 205 -> 188, 1024 428 both (the column-per-wavefront kernel 127, 147, 250, 603)
    const bool short_k = R > 512 && K <= 1024;
    // Quantised matrices: 96 where that is all of them, beyond it the cost chooses among blocks of 80, 96 and 128
    // (int4 of a few groups: 96 beyond 48 rows as well, where the wavefronts share K two ways, not four.  80 rows, a layer of d_model 128 | 256 | 512, us: QKV in
    // 80 -> 96 rows 42.8 -> 41.2 | 45.2 -> 43.5 | 51.1 -> 49.9, gate and up another 0.6 | 0.6 | 0.1 less)
    const bool few_groups = bits == 4 && fused && K <= 512 && R > 48;
    const int q0 = R <= 32 ? 32 : R <= 48 ? 48 : R <= 80 && !few_groups ? 80 : 96, q1 = R <= 96 ? q0 : 128;
    const int rows[5] = {32, 48, 80, 96, 128}, narrow[4] = {64, 96, 128, 192}, plain[2] = {64, 128};
    const int splits = epi == EPI_QKV ? 4 : epi == EPI_RESID ? 8 : 1;
    TileChoice best{0, 0, 1, 1e30};
    for (int bm : rows) {
        if (bits == 16 ? bm != bm0 && !(short_k && bm < bm0 && bm != 96) : bm > q1 || (bm < (few_groups ? 96 : std::min(q0, 80)) && !short_k)) continue;
        for (int i = 0; i < (fused ? 4 : 2); ++i) {
            const int cols = fused ? narrow[i] : plain[i];
            if (bm >= 96 && cols == 64 && (fused || bits < 16)) continue;
            if (bits < 16 && fused && cols == 64) continue;
            // Gate and up in 128 columns: one row block, where 96 columns make more workgroups than there are compute units and 128 do not.  192, the other
            // way to one round, leave up to half of the units idle: 13B shape, 27648 columns, 144 workgroups of 192 -> 216 of 128, a layer, us: bf16
            // 18 | 40 | 80 rows 156.3 -> 147.9 | 180.5 -> 167.7 | 218.4 -> 205.0; two of int8 240.6 -> 224.7 | 289.8 -> 274.5 | 391.6 -> 372.2; three of
            // int4 404.0 -> 375.0 | 478.4 -> 449.9 | 646.6 -> 603.3.  (QKV splits K instead: level with 192 columns by the cost.)
            if (fused && cols == 128 && (epi == EPI_QKV || bm > 80 || R > bm || (columns + 95) / 96 <= 256 || (columns + 127) / 128 > 256)) continue;
            for (int ks = 1; ks <= splits; ++ks) {
                // (Quantised, K between 256 and 512: shares of a stage or two cost more than they save.  A layer of d_model 128, d_ff 384, 18 rows, three
                // shares -> one: int4 32.2 -> 30.7 us, int8 32.1 -> 30.4.)
                if (ks > 1 && (sizeof(float) * (size_t)ks * R * N > ws_bytes || (short_k && K < 256 * ks) || (bits < 16 && K > 256 && K < 512))) break;
                const TileChoice c = tile_cost(epi, bits, bm, cols, columns, R, K, ks, epi == EPI_QKV ? 4.5 : 0.0, short_k);
                if (c.us < best.us) best = c;
            }
        }
    }
    return best;
}
template <int EPI, int QB> static int launch_tile(const GemmArgs &a, int tiles, hipStream_t st) {
    const int columns = 16 * tiles * (EPI == EPI_SWIGLU || EPI == EPI_QKV ? 2 : 1);
    // partial rows need whole 16-column tiles, room in the workspace and, for a residual, dense output rows
    const bool split_ok = a.splitk_ws && a.N % 16 == 0 && (EPI == EPI_QKV || (EPI == EPI_RESID && a.ldo == a.N && a.out == a.resid));
    const TileChoice best = choose_tile(EPI, QB ? QB : 16, tiles, a.R, a.N, a.K, split_ok ? a.splitk_ws_bytes : 0);
    return launch_tile_as_chosen<EPI, QB>(a, columns, best, st);
}
// For the tests, which have to meet every tile (not part of the library's interface): what a launch of R rows, N columns (3 * heads *
// head_dim for EPI_QKV) and K entries takes: rows and columns of a workgroup, splits of K.
extern "C" void ss_dev_gemm_tile_bits(int bits, int epi, int R, int N, int K, size_t ws_bytes, int *out3) { // bits 16, 8 or 4
    const TileChoice c = choose_tile(epi, bits, epi == EPI_QKV ? N / 32 : (N + 15) / 16, R, N, K, N % 16 == 0 ? ws_bytes : 0);
    out3[0] = c.rows; out3[1] = c.cols; out3[2] = c.ksplit;
}
extern "C" void ss_dev_gemm_tile(int epi, int R, int N, int K, size_t ws_bytes, int *out3) { ss_dev_gemm_tile_bits(16, epi, R, N, K, ws_bytes, out3); }

// Calls of at most 16 rows.  The output columns in quads (of pairs for the fused epilogues) over k workgroups per compute unit of at
// most eight quads, every one with the same number or one more: the smallest k - except that up to 8 rows a k that makes a tenth fewer
// 16-column tiles of them is taken (a tile costs its LDS reads, MFMAs and conversions whether it is full or not: 2752 quads of pairs, K 4096,
// three workgroups of four at most against two of six, one tile and a half: 28.8 against 29.2 us bf16, 18.5 / 20.3 int8, 14.5 / 16.6 int4).
// Fewer tiles than that don't pay for the workgroups (heads of 50257 columns, 13 tiles against 14 but 13 workgroups against 7, 5 rows, us:
// K 256 bf16 16.6 / 15.6, K 4096 73.8 / 71.4, int8 52.6 / 48.0, int4 42.6 / 36.4; K 256 fp32 18.4 / 19.4), nor beyond 8 rows, where
// every workgroup's activations weigh as much as its weights (12 rows: 31.2 us with two, 32.6 with three).
struct ColumnSplit {
    int groups, quads, rest; // workgroups; quads of each, and one more in the first `rest`
};
static ColumnSplit split_columns(int epi, int N, int R) {
    constexpr int UNITS = 256;
    const int quads = epi == EPI_QKV ? N / 8 : (N + 3) / 4;
    auto tiles = [&](int k) { return k * (((quads + UNITS * k - 1) / (UNITS * k) + 3) / 4); };
    const int least = (quads + UNITS * 8 - 1) / (UNITS * 8);
    int k = least;
    for (int i = least + 1; R <= 8 && i <= 2 * least; ++i)
        if (10 * tiles(i) < 9 * tiles(k)) k = i;
    const int groups = std::min(quads, k * UNITS);
    return ColumnSplit{groups, quads / groups, quads % groups};
}
int deferred_norm_parts(int d) {
    const int groups = split_columns(EPI_RESID, d, 1).groups;
    return d % 4 == 0 && groups % 16 == 0 && groups <= NSQ_MAX_PARTS ? groups : 0; // (at most 256 workgroups: one k whatever the rows)
}
// For the tests, which have to meet every size (not part of the library's interface): workgroups, quads of each, workgroups with one more.
extern "C" void ss_dev_gemm_share(int epi, int R, int N, int *out3) {
    const ColumnSplit s = split_columns(epi, N, R);
    out3[0] = s.groups; out3[1] = s.quads; out3[2] = s.rest;
}
template <typename T, int QB, int EPI, int NW, int NB, int EI, int RCAP>
static void launch_cols_as(const GemmArgs &a0, const ColumnSplit &s, hipStream_t st) {
    GemmArgs a = a0;
    a.quads = s.quads; a.quads_rest = s.rest; a.nsq_parts = s.groups;
    hipLaunchKernelGGL((gemm_cols_kernel<T, QB, EPI, NW, NB, EI, RCAP>), dim3(s.groups), dim3(NW * 64), 0, st, a);
}
// Wavefronts and buffers, from all of (2 .. 16 waves) x (1, 2 buffers) on the matrices of four decoder widths (2048 - 5120) at 1, 5, 12 and 16
// rows, within 3 % of the best for each: 60 - 90 KB asked for per compute unit (a unit has some 32 KB in flight; more only delays what
// is needed first), by few waves with two buffers where steps are long and by many with one where they are short.  many: several
// workgroups per compute unit.
struct Ring {
    int waves, buffers;
};
constexpr Ring ring_for(int bits, int epi, int ei, int rcap, bool many) {
    const bool resid = epi == EPI_RESID, store = epi == EPI_STORE;
    if (bits == 4) {
        if (rcap == 16) return resid ? (ei <= 3 ? Ring{8, 1} : Ring{6, 1}) : !many && ei <= 2 ? Ring{4, 1} : Ring{6, 1};
        return resid ? Ring{12, 1} : many ? Ring{4, 1} : Ring{8, 1};
    }
    if (bits == 8) {
        if (rcap == 16) return resid ? Ring{12, 1} : many ? Ring{4, 1} : Ring{8, 1};
        if (many) return store ? Ring{2, 2} : Ring{4, 1};
        return resid ? Ring{8, 2} : ei <= 2 ? Ring{8, 1} : ei == 3 ? Ring{12, 1} : Ring{4, 2};
    }
    if (many) return store || (rcap == 8 && ei > 2) ? Ring{4, 2} : Ring{4, 1};
    if (resid || store) return Ring{8, 2};
    if (ei <= 2) return rcap == 16 ? Ring{12, 1} : Ring{8, 1};
    return ei == 3 || rcap == 16 ? Ring{6, 2} : Ring{4, 2};
}
template <typename T, int QB, int EPI, int EI, bool MANY, int RCAP> static void launch_cols_rows(const GemmArgs &a, const ColumnSplit &s, hipStream_t st) {
    constexpr Ring RING = ring_for(QB ? QB : 8 * (int)sizeof(T), EPI, EI, RCAP, MANY);
    if (QB == 4 && RCAP == 8 && a.R <= 5) launch_cols_as<T, QB, EPI, RING.waves, RING.buffers, EI, QB == 4 && RCAP == 8 ? 5 : RCAP>(a, s, st); // (a step of int4 is mostly activations)
    else launch_cols_as<T, QB, EPI, RING.waves, RING.buffers, EI, RCAP>(a, s, st);
}
template <typename T, int QB, int EPI, int EI> static void launch_cols_ei(const GemmArgs &a, const ColumnSplit &s, hipStream_t st) {
    if (a.R <= 8) launch_cols_rows<T, QB, EPI, EI, false, 8>(a, s, st);
    else launch_cols_rows<T, QB, EPI, EI, false, 16>(a, s, st);
}
template <typename T, int QB, int EPI> static int launch_cols(const GemmArgs &a, hipStream_t st) {
    const ColumnSplit s = split_columns(EPI, a.N, a.R);
    const int ei = (s.quads + (s.rest ? 1 : 0) + 1) / 2;
    constexpr bool M = EPI != EPI_RESID; // (a residual's columns fill more than one workgroup per unit beyond 8192 only)
    if (M && s.groups > 256) { // shares of up to 4 and of 7 or 8 quads up to 8 rows, of 5 or 6 and of 7 or 8 beyond: split_columns makes no others
        if (a.R <= 8) {
            if (ei <= 2) launch_cols_rows<T, QB, EPI, 2, M, 8>(a, s, st);
            else launch_cols_rows<T, QB, EPI, 4, M, 8>(a, s, st);
        } else {
            if (ei <= 3) launch_cols_rows<T, QB, EPI, 3, M, 16>(a, s, st);
            else launch_cols_rows<T, QB, EPI, 4, M, 16>(a, s, st);
        }
    } else if (ei == 1) {
        launch_cols_ei<T, QB, EPI, 1>(a, s, st);
    } else if (ei == 2) {
        launch_cols_ei<T, QB, EPI, 2>(a, s, st);
    } else if (ei == 3) {
        launch_cols_ei<T, QB, EPI, 3>(a, s, st);
    } else {
        launch_cols_ei<T, QB, EPI, 4>(a, s, st);
    }
    return (EPI == EPI_RESID && a.nsq_out) ? 2 : 0;
}

template <int EPI> static int launch_wide_any(const GemmArgs &a, int tiles, int row_tiles, hipStream_t st) {
    // larger batches and prefill chunks: waves split the columns; fewer waves per workgroup when the
    // matrix has few tiles, so that the launch still covers the chip
    constexpr bool FUSED = EPI == EPI_SWIGLU || EPI == EPI_QKV; // two weight tiles per wave: more registers
    const bool small = tiles < 8 * 128;
    if (row_tiles <= 2) {
        if (small) return launch_wide<EPI, 4, 2>(a, tiles, row_tiles, st);
        return launch_wide<EPI, 8, 2>(a, tiles, row_tiles, st);
    } else if (row_tiles <= 3) {
        if (small) return launch_wide<EPI, 4, 3>(a, tiles, row_tiles, st);
        return launch_wide<EPI, 8, 3>(a, tiles, row_tiles, st);
    } else {
        // one workgroup per compute unit fits: 3 waves per workgroup when that fills more of a 256-unit chip
        // in whole rounds than 4 (688 gate/up tiles: 230 workgroups instead of 172; 384 QKV tiles: 128, split in two)
        auto fill = [&](int nw) {
            const int wgs = (tiles + nw - 1) / nw * ((row_tiles + 4) / 5);
            const int ks = std::max(1, std::min(256 / std::max(wgs, 1), 4));
            return (double)(wgs * ks) / (double)((wgs * ks + 255) / 256 * 256);
        };
        if constexpr (!FUSED) {
            if (!small) return launch_wide<EPI, 8, 5>(a, tiles, row_tiles, st);
        }
        if (fill(3) > fill(4) + 0.1) return launch_wide<EPI, 3, 5>(a, tiles, row_tiles, st);
        return launch_wide<EPI, 4, 5>(a, tiles, row_tiles, st);
    }
}

template <typename T, int QB, int EPI> static int launch_gemm_t(const GemmArgs &a, hipStream_t st) {
    const int row_tiles = (a.R + 15) / 16;
    if (row_tiles <= 1) return launch_cols<T, QB, EPI>(a, st);
    const int tiles = EPI == EPI_QKV ? 3 * a.H * (a.hd / 32) : (a.N + 15) / 16;
    if constexpr (std::is_same<T, bf16_t>::value) return launch_tile<EPI, QB>(a, tiles, st);
    else return launch_wide_any<EPI>(a, tiles, row_tiles, st);
}

int launch_gemm(int dtype, int epi, const GemmArgs &a, hipStream_t st) {
    // quantised weights: the caller has checked bf16 planes and K % 128 == 0 (int4) or K % 16 == 0 (int8)
    const int kind = a.wscale ? a.wbits : dtype ? 16 : 32;
#define SS_CASE(EP)                                              \
    case EP:                                                     \
        return kind == 4   ? launch_gemm_t<bf16_t, 4, EP>(a, st)   \
               : kind == 8  ? launch_gemm_t<bf16_t, 8, EP>(a, st)  \
               : kind == 16 ? launch_gemm_t<bf16_t, 0, EP>(a, st)  \
                            : launch_gemm_t<float, 0, EP>(a, st);
    switch (epi) {
        SS_CASE(EPI_STORE)
        SS_CASE(EPI_RESID)
        SS_CASE(EPI_SWIGLU)
        SS_CASE(EPI_QKV)
    }
#undef SS_CASE
    return 0;
}

} // namespace ss
