// Tetra matrix times many activation rows (a prompt, Sec. 6: the served
// model runs a prompt in one call): decode on the vector unit, products on
// the matrix cores.  Included by tetra.hip after kernels.h.
//
// y[n][row] = sigma_row * sum_blk s_blk * sum_j y_j x[n][24 blk + j]
//             + sum_t tail_t x[n][24 nblk + t]
//
// is the same sum as the GEMV's.  The decoded y_j are exact integers in fp16;
// the block's scale is folded into them as fp16(s_blk y_j), rounded once from
// the fp32 product, so that the matrix cores accumulate straight into the
// sums across blocks; sigma and the tail are applied at the end.  The fold
// costs one rounding of each weight to fp16: a relative error of at most
// 2^-11 per weight, so at most 2^-11 (4.9e-4) of sum |w x| per output, inside
// the 1e-3 bound of the products (the GEMV keeps the scale in fp32).
//
// MFMA roles (v_mfma_f32_32x32x16_f16): A = activations (32 tokens x 16 k),
// B = decoded weights (16 k x 32 rows), D = 32 tokens x 32 rows.  Lane l
// holds A[l % 32][8h..8h+7] and B[8h..8h+7][l % 32] with h = l / 32, and
// D[8g + 4h + r][l % 32] in register 4g + r.  Blocks go in pairs, a window of
// 48 k: the lanes of half h decode block h of the pair, one row each, and
// product kk (of three) takes section kk of both blocks.  So every lane
// decodes one whole block of its own per window, without any exchange between
// lanes, and gets all of its row's block scale; the activations are laid out
// to match.
//
// A workgroup of eight waves takes up to 256 tokens (TG groups of 32) and a
// wave 32 rows by all of them, so that each decoded block feeds TG x 3
// products.  Two waves share a SIMD (128 accumulators each): one wave alone
// (64 rows, 512 registers) issues an instruction every five cycles at most
// and was bound by that, 0.445 ms where this form takes 0.435 (12288 x 4096 by
// 4096 tokens) and 2.7 us a chunk where it takes 2.3 (20 workgroups).  With S =
// 1 the waves hold 8 x 32 rows; with S = 2 they hold 4 x 32 rows, and two waves
// share a row set, one for each window of a chunk, their sums meeting in LDS at
// the end: half the rows per workgroup, for launches that must be cut into
// pieces to fill the chip (a piece then is half as large).
//
// The activations go through LDS in chunks of 96 k (one group of four block
// columns), double-buffered, one barrier per chunk: the next chunk's are
// loaded into registers during the first half of a chunk and written to the
// other buffer during the second.  The decode of the next window is placed
// between the products of the present one, step by step (pf_step), since the
// compiler's own order puts the products first and the decode after them.
//
// Work split with S = 2 (stream-K): an item is a (row group, token tile) and
// a unit is one chunk of an item (the trailing block columns of a row make
// one more, shorter unit).  The workgroups (one per CU, fewer for few items)
// take equal contiguous ranges of the items' units.  Of an item whose units
// span several workgroups each stores its sums in the workspace, and a second
// kernel on the whole chip (gemm_sum_kernel) adds the pieces in workgroup
// order, which makes the result independent of timing.  (The last workgroup
// of an item to finish adding them by itself took as long as the product:
// 1024 x 5120 by 203 tokens 39 us against 22, 5120 x 5120 52 against 37.)
// With S = 1 every workgroup takes whole items.
//
// Measured against a kernel of four waves with 32x32x8 products, each lane
// decoding half a block, at two workgroups per CU: 12288 x 4096 by 4096
// tokens 0.86 -> 0.42 ms (992 TFLOP/s, the clock then at 1.8 to 1.9 GHz: the
// chip is at its power limit), 17408 x 5120 by 203 tokens 125 -> 71 us.
#pragma once

#include <type_traits>
#include <utility>

namespace tetra_dev {

constexpr int kPfWaves = 8;
constexpr int kPfThreads = kPfWaves * 64;
constexpr int kPfChunk = 96;               // k per chunk: four blocks, two windows
constexpr int kPfMaxTG = 8;                // 32-token groups of a workgroup, at most
constexpr int kPfGroupsPerCU = 1;          // 54 KB of tables, up to 96 KB of activations
constexpr int kPfFrag = 1024;              // bytes of one A operand (32 tokens x 16 k) in LDS

// floats of one workgroup's piece of an item (128 rows by 256 tokens)
constexpr int kPfSlot = 128 * 32 * kPfMaxTG;

struct GemmArgs {
    const uint8_t* codes;
    const uint16_t* sigma;
    const uint16_t* x;                     // [N][K] fp16
    float* y;                              // [N][M]
    unsigned long long tail_off;
    int M, K, N, nblk, T, ng, rem;
    int tgroups;                           // token tiles
    int tiles;                             // 64-row tiles
    int upi;                               // units per item: ng, plus one when rem > 0
    int items;
    int workers;                           // workgroups of the launch
    unsigned long long units;              // items * upi
    float* partials;                       // [workers][2][kPfSlot]
};

typedef uint32_t pf_u32x4 __attribute__((ext_vector_type(4)));

// a buffer of `bytes` from p (the same for the whole wave): loads from it
// take a 32-bit lane offset and a scalar one
constexpr int kPfRsrcWord3 = 0x00020000;   // raw 32-bit buffer, gfx9
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pf_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), static_cast<short>(0), static_cast<int>(bytes),
                                             kPfRsrcWord3);
}

// Values pass through these helpers by value: __builtin_bit_cast applied
// directly to a subscript of a vector (acc[tg][i], q[i]) was compiled as a
// cast of element 0 whatever i was.
__device__ __forceinline__ uint32_t pf_bits(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ __forceinline__ float pf_float(uint32_t u) { return __builtin_bit_cast(float, u); }

// component i (a constant) of a quad
__device__ __forceinline__ uint32_t pf_part(const pf_u32x4& v, int i) {
    return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
}

// workspace of a launch with at most `workers` workgroups: eight bytes each,
// rounded up to 256, that hold nothing (kept so that the sizes callers have
// allocated go on holding the same pieces), then two piece slots per workgroup
inline size_t gemm_header_bytes(int workers) {
    return (8 * static_cast<size_t>(workers) + 255) & ~static_cast<size_t>(255);
}
inline size_t gemm_workspace_bytes(int workers) {
    return gemm_header_bytes(workers) + sizeof(float) * static_cast<size_t>(workers) * 2 * kPfSlot;
}

// a workgroup-uniform 64-bit value in scalar registers (the 64-bit divisions
// below run on the vector unit, which would leave every index derived from
// them, and the loops they bound, in vector registers)
__device__ __forceinline__ unsigned long long pf_uniform(unsigned long long v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// first unit of workgroup w's range (w = workers gives the end)
__device__ __forceinline__ unsigned long long pf_range_begin(int w, const GemmArgs& a) {
    return pf_uniform(a.units * static_cast<unsigned long long>(w) / static_cast<unsigned long long>(a.workers));
}

// the workgroup whose range holds unit u
__device__ __forceinline__ int pf_worker_of(unsigned long long u, const GemmArgs& a) {
    return __builtin_amdgcn_readfirstlane(
        static_cast<int>(((u + 1) * static_cast<unsigned long long>(a.workers) - 1) / a.units));
}

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));

// f(constant 0) .. f(constant N - 1): the product loop is unrolled by the
// front end (the optimizer gives up on loops of this size)
template <int... I, class F>
__device__ __forceinline__ void pf_for_impl(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void pf_for(F&& f) {
    pf_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// this thread's index in the workgroup, read afresh at each use: an index
// derived from threadIdx once would stay in a register across the whole
// item loop
__device__ __forceinline__ int pf_tid() {
    return (__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x)) & ~63) | lane_now();
}

// the B operands of a window (three 16-k steps): this lane's block
struct PfBlock {
    pf_u32x4 b[3];
};

// the decode of a block in flight
struct PfDecode {
    uint32_t e, r[6], pm, a1, am, u3, ep, qp, sg, y[12];
    float sa, sb, s, t[4];
};

// The decode of one block per lane (word lo, hi) as kPfSteps steps of a few
// instructions each: the table reads, the values with their norm (as
// fetch_block and block_values form them), the scale's read, and the values
// times the scale, rounded once from the fp32 product.  v_fma_mix_f32 twice
// and one v_cvt_pk_f16_f32 per pair: the mixed fmas that write half a
// register (v_fma_mixlo / mixhi) take 8.6 cycles each against 5.3, so the
// pair is kept from being formed that way.
constexpr int kPfSteps = 5 + 24 + 1 + 18;

template <int n>
__device__ __forceinline__ void pf_step(PfDecode& d, PfBlock& o, uint32_t lo, uint32_t hi, lds_bytes* L) {
    if constexpr (n == 0) {
        d.e = *(lds_u32*)(L + kPathOff + ((lo << 2) & 0x3FFCu));                 // 4 * path
        uint32_t i2 = __builtin_amdgcn_alignbit(hi, lo, 25) & 0x7FFu;
        asm("" : "+v"(i2));
        d.am = i2 * 8u + 8u * tetra::kMidOffset;                                 // 8 * (808 + i2), bit 14 = delta
        asm("" : "+v"(d.am));
    } else if constexpr (n == 1) {
        d.a1 = (lo >> 10) & 0x7FF8u;                                             // 8 * phys1
        const u32x2 r1 = *(lds_u2*)(L + kRowsOff + d.am);
        const u32x2 r0 = *(lds_u2*)(L + kRowsOff + d.a1);
        d.r[0] = r0.x;
        d.r[1] = r0.y;
        d.r[2] = r1.x;
        d.r[3] = r1.y;
    } else if constexpr (n == 2) {
        d.u3 = (hi >> 1) & 0x7FF8u;                                              // 8 * ((p ^ r) << 11 | i3')
        const uint32_t a3 = d.u3 ^ (d.am & 0x4000u);                             // 8 * phys3 (Eq. 3)
        const u32x2 r2 = *(lds_u2*)(L + kRowsOff + a3);
        d.r[4] = r2.x;
        d.r[5] = r2.y;
    } else if constexpr (n == 3) {
        d.pm = static_cast<uint32_t>(static_cast<int32_t>((d.a1 ^ d.u3) << 17) >> 31);   // p = r ^ (p ^ r)
        d.sa = pf_float((lo & 0x1000u) | 0x4B000000u);                           // 2^23 + 4096 g
        d.sb = 0.f;
    } else if constexpr (n == 4) {
        d.ep = d.e ^ (~d.pm & 0xFCFCFCFCu);
        d.qp = ~d.pm & 0x3C003C00u;
    } else if constexpr (n < 29) {
        constexpr int k = (n - 5) >> 2, q = (n - 5) & 3;
        if constexpr (q == 0) {
            d.sg = d.r[k] ^ ((d.ep << k) & 0x80808080u);
        } else if constexpr (q == 1) {
            d.y[2 * k] = cvt_pair<false>(d.sg);
            d.y[2 * k + 1] = cvt_pair<true>(d.sg);
        } else if constexpr (q == 2) {
            d.y[2 * k] = pk_add(d.y[2 * k], d.qp);
            d.y[2 * k + 1] = pk_add(d.y[2 * k + 1], d.qp);
        } else {
            d.sa = dot2(d.y[2 * k], d.y[2 * k], d.sa);
            d.sb = dot2(d.y[2 * k + 1], d.y[2 * k + 1], d.sb);
        }
    } else if constexpr (n == 29) {
        d.s = *(lds_f32*)(L + kScaleOff + ((pf_bits(d.sa + d.sb) >> 2) & 0x7FFu));
    } else {
        constexpr int k = (n - 30) / 3, q = (n - 30) % 3;
        if constexpr (q < 2) {
            const half2_t h = __builtin_bit_cast(half2_t, d.y[2 * k + q]);
            float u = __builtin_fmaf(static_cast<float>(h[0]), d.s, 0.f);
            float v = __builtin_fmaf(static_cast<float>(h[1]), d.s, 0.f);
            asm("" : "+v"(u));
            asm("" : "+v"(v));
            d.t[2 * q] = u;
            d.t[2 * q + 1] = v;
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                half2_t v;
                v[0] = static_cast<_Float16>(d.t[2 * i]);
                v[1] = static_cast<_Float16>(d.t[2 * i + 1]);
                o.b[(2 * k + i) >> 2][(2 * k + i) & 3] = __builtin_bit_cast(uint32_t, v);
            }
        }
    }
}

// a lane's code words of a chunk: its row's block 2j + h for the windows j
struct PfWords {
    uint32_t lo[2], hi[2];
};

// a chunk of the activations in flight: a token's 192 bytes are twelve
// 16-byte pieces; a thread holds pieces xq, xq + 4 and xq + 8 of one token in
// every 128, so that four threads read 64 bytes of a token at once
template <int TG>
struct PfX {
    static constexpr int kIt = (TG + 3) / 4;
    typedef uint32_t vec_t __attribute__((ext_vector_type(12 * kIt)));
    vec_t v;
};

// LDS bytes of a chunk buffer: fragments [token group][window][kk], token
// groups in fours; two of them also take the sums that waves exchange
template <int TG>
constexpr int pf_buf_bytes() {
    return (TG + 3) / 4 * 4 * 6 * kPfFrag;
}

template <int TG, int S>
__global__ __launch_bounds__(kPfThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_kernel(const GemmArgs a) {
    static_assert(S == 1 || S == 2, "windows of a chunk per wave: two or one");
    __shared__ uint4 s_tab[kPackedTableBytes / 16];
    __shared__ __attribute__((aligned(16))) uint8_t s_x[2][pf_buf_bytes<TG>()];
    TableStage<kPfThreads> ts;
    ts.load();                                             // stored below, after the ranges are worked out
    lds_bytes* L = (lds_bytes*)(s_tab);
    constexpr int kRowSets = kPfWaves / S;                 // 32-row sets of a workgroup
    constexpr int kSlots = 3 * TG;                         // products of a window
    constexpr int kAhead = 3;                              // A operands read ahead
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int rset = S == 1 ? wave : wave >> 1, ksplit = S == 1 ? 0 : wave & 1;
    const int lane = threadIdx.x & 63, h = lane >> 5, jr = lane & 31;
    // LDS byte of this lane's A operand of product kk in window j (S = 2: in
    // this wave's window), piece q = 6 j + 3 h + kk of its token: the tokens
    // of a half fragment are permuted by 4 (q mod 4), so that neither the
    // reads (16 lanes of a half at once) nor the writes (four pieces of four
    // tokens) meet in a bank
    uint32_t ar[2][3];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int kk = 0; kk < 3; ++kk) {
            const int jj = S == 2 ? ksplit : j;
            ar[j][kk] = static_cast<uint32_t>((3 * jj + kk) * kPfFrag + 512 * h +
                                              16 * (jr ^ (4 * ((6 * jj + 3 * h + kk) & 3))));
        }
    // this thread's pieces of a chunk: xq + 4 i of token xtok + 128 it
    const int xtok = threadIdx.x >> 2, xq = threadIdx.x & 3;
    uint32_t xl[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int q = xq + 4 * i, b = q / 3, kk = q - 3 * b;
        xl[i] = static_cast<uint32_t>(((xtok >> 5) * 6 + 3 * (b >> 1) + kk) * kPfFrag + 512 * (b & 1) +
                                      16 * ((xtok & 31) ^ (4 * xq)));
    }
    const uint32_t wlo = static_cast<uint32_t>(16 * (32 * (rset & 1) + jr) + 4 * h + 8 * ksplit);
    const uint32_t whi = static_cast<uint32_t>(1024 + 8 * (32 * (rset & 1) + jr) + 2 * h + 4 * ksplit);
    const __amdgpu_buffer_rsrc_t xrs = pf_rsrc(a.x, static_cast<uint32_t>(2 * a.K) * static_cast<uint32_t>(a.N));
    float16_t acc[TG];

    const unsigned long long u0 = S == 1 ? 0 : pf_range_begin(blockIdx.x, a);
    const unsigned long long u1 = S == 1 ? 0 : pf_range_begin(blockIdx.x + 1, a);
    unsigned long long base = S == 1 ? 0 : pf_uniform(u0 - u0 % a.upi);
    ts.store(s_tab);
    for (int item = S == 1 ? static_cast<int>(blockIdx.x)
                           : __builtin_amdgcn_readfirstlane(static_cast<int>(base / a.upi));
         S == 1 ? item < a.items : base < u1; item += S == 1 ? a.workers : 1, base += a.upi) {
        // this workgroup's units c0 .. c1-1 of the item
        const int c0 = S == 1 ? 0 : __builtin_amdgcn_readfirstlane(static_cast<int>((u0 > base ? u0 : base) - base));
        const unsigned long long last = u1 < base + a.upi ? u1 : base + a.upi;
        const int c1 = S == 1 ? a.upi : __builtin_amdgcn_readfirstlane(static_cast<int>(last - base));
        const int irow = item / a.tgroups;
        const int n0 = (item - irow * a.tgroups) * (32 * TG);
        // the wave's row set; past the last tile it repeats that and stores nothing
        const int wt_raw = (irow * kRowSets + rset) >> 1;
        const int wt = min(wt_raw, a.tiles - 1);
        const uint8_t* tb = a.codes + static_cast<size_t>(wt) * a.nblk * kChunk;
        const __amdgpu_buffer_rsrc_t tr = pf_rsrc(tb, static_cast<uint32_t>(a.nblk) * kChunk);
        uint32_t xg[PfX<TG>::kIt];                         // tokens past N read row N - 1: never stored
#pragma unroll
        for (int it = 0; it < PfX<TG>::kIt; ++it)
            xg[it] = static_cast<uint32_t>(min(n0 + 128 * it + xtok, a.N - 1)) * static_cast<uint32_t>(2 * a.K) + 16u * xq;
        constexpr int kPieces = 3 * PfX<TG>::kIt;
        PfX<TG> xr;
        PfWords wc, wn;
        // chunk c; the trailing columns (c = ng) are zero past the last block,
        // and their words past it decode to the origin
        auto load_x = [&](int c) {
            auto get = [&](auto p, uint32_t at) {
                const pf_u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(xrs, at, 2 * kPfChunk * c, 0);
                xr.v[4 * p] = q.x;
                xr.v[4 * p + 1] = q.y;
                xr.v[4 * p + 2] = q.z;
                xr.v[4 * p + 3] = q.w;
            };
            if (c < a.ng)
                pf_for<kPieces>([&](auto p) { get(p, xg[p / 3] + 64 * (p % 3)); });
            else                                           // past the last block: out of the buffer, which reads zero
                pf_for<kPieces>([&](auto p) {
                    get(p, xq + 4 * (p % 3) < 3 * a.rem ? xg[p / 3] + 64 * (p % 3) : 0x80000000u);
                });
        };
        auto store_x = [&](uint8_t* dst, auto p) {         // piece p % 3 of token xtok + 128 (p / 3)
            *reinterpret_cast<uint4*>(dst + xl[p % 3] + 24 * (p / 3) * kPfFrag) =
                make_uint4(xr.v[4 * p], xr.v[4 * p + 1], xr.v[4 * p + 2], xr.v[4 * p + 3]);
        };
        auto load_w = [&](PfWords& w, int c) {
            if (c < a.ng) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if (S == 2 && j == 1) continue;
                    w.lo[j] = __builtin_amdgcn_raw_buffer_load_b32(tr, wlo + 8 * j, c * tetra::kGroupBytes, 0);
                    w.hi[j] = static_cast<uint16_t>(
                        __builtin_amdgcn_raw_buffer_load_b16(tr, whi + 4 * j, c * tetra::kGroupBytes, 0));
                }
            } else {
                const int ln = lane_now();
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if (S == 2 && j == 1) continue;
                    const int q = 2 * (S == 2 ? ksplit : j) + (ln >> 5);
                    const int col = 4 * a.ng + min(q, a.rem - 1);
                    const tetra::WordLoc at = tetra::word_loc(a.nblk, 32 * (rset & 1) + (ln & 31), col);
                    w.lo[j] = *reinterpret_cast<const uint32_t*>(tb + at.lo_off);
                    w.hi[j] = *reinterpret_cast<const uint16_t*>(tb + at.hi_off);
                    if (q >= a.rem) {
                        w.lo[j] = tetra::kZeroLo;
                        w.hi[j] = tetra::kZeroHi;
                    }
                }
            }
        };
        PfDecode d;
        PfBlock ba, bb;
        half8_t av[kAhead + 1];
        auto frag = [&](const uint8_t* xs, const uint32_t (&at)[3], int slot) {
            return *reinterpret_cast<const half8_t*>(xs + at[slot / TG] + 6 * (slot % TG) * kPfFrag);
        };
        // the products of the window at `at` of the chunk xs with `cur`, and
        // between them the decode of the words lo, hi into `nxt`
        auto window = [&](const uint8_t* xs, const uint32_t (&at)[3], const PfBlock& cur, PfBlock& nxt, uint32_t lo,
                          uint32_t hi, auto&& also) {
            pf_for<kAhead>([&](auto s) {
                if constexpr (s < kSlots) av[s] = frag(xs, at, s);
            });
            pf_for<kSlots>([&](auto s) {
                if constexpr (s + kAhead < kSlots) av[(s + kAhead) % (kAhead + 1)] = frag(xs, at, s + kAhead);
                acc[s % TG] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                    av[s % (kAhead + 1)], __builtin_bit_cast(half8_t, cur.b[s / TG]), acc[s % TG], 0, 0, 0);
                also(s);
                constexpr int i0 = s * kPfSteps / kSlots, i1 = (s + 1) * kPfSteps / kSlots;
                pf_for<i1 - i0>([&](auto i) { pf_step<i0 + i>(d, nxt, lo, hi, L); });
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        // the stores of the next chunk spread over a window's second part
        auto put_next = [&](uint8_t* dst, auto s) {
            constexpr int first = kSlots / 2;
            constexpr int p0 = s < first ? 0 : (s - first) * kPieces / (kSlots - first);
            constexpr int p1 = s < first ? 0 : (s + 1 - first) * kPieces / (kSlots - first);
            pf_for<p1 - p0>([&](auto p) { store_x(dst, std::integral_constant<int, p0 + p>{}); });
        };

#pragma unroll
        for (int t = 0; t < TG; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
        load_w(wc, c0);
        load_x(c0);
        __syncthreads();                                   // tables staged; LDS of the previous item read
        pf_for<kPieces>([&](auto p) { store_x(s_x[c0 & 1], p); });
        pf_for<kPfSteps>([&](auto i) { pf_step<i>(d, ba, wc.lo[0], wc.hi[0], L); });
        __syncthreads();
        for (int c = c0; c < c1; ++c) {
            const uint8_t* xs = s_x[c & 1];
            uint8_t* dst = s_x[(c & 1) ^ 1];
            const int cn = min(c + 1, c1 - 1);             // past the last: it again, not used
            load_w(wn, cn);
            load_x(cn);
            if constexpr (S == 1) {
                window(xs, ar[0], ba, bb, wc.lo[1], wc.hi[1], [&](auto) {});
                window(xs, ar[1], bb, ba, wn.lo[0], wn.hi[0], [&](auto s) { put_next(dst, s); });
            } else {
                window(xs, ar[0], ba, bb, wn.lo[0], wn.hi[0], [&](auto s) { put_next(dst, s); });
                ba = bb;
            }
            wc = wn;
            __syncthreads();
        }

        // S = 2: the two waves of a row set add their sums, the first TH token
        // groups in the one and the others in the other
        constexpr int TH = S == 1 ? TG : (TG + 1) / 2;
        const int t0 = S == 1 ? 0 : ksplit * TH;           // first of this wave's token groups, then in acc[0 .. TH-1]
        if constexpr (S == 2) {
            pf_u32x4* ex = reinterpret_cast<pf_u32x4*>(s_x[0]) + rset * (TH * 256) + lane_now();
            static_assert(kPfWaves / 2 * TH * 4096 <= 2 * pf_buf_bytes<TG>(), "exchange fits the chunk buffers");
            auto give = [&](auto first) {
                pf_for<TH>([&](auto t) {
                    if constexpr (first + t < TG)
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            ex[(4 * t + k) * 64] =
                                pf_u32x4{pf_bits(acc[first + t][4 * k]), pf_bits(acc[first + t][4 * k + 1]),
                                         pf_bits(acc[first + t][4 * k + 2]), pf_bits(acc[first + t][4 * k + 3])};
                });
            };
            auto take = [&](auto first) {
                pf_for<TH>([&](auto t) {
                    if constexpr (first + t < TG)
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const pf_u32x4 o = ex[(4 * t + k) * 64];
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                acc[t][4 * k + i] = acc[first + t][4 * k + i] + pf_float(pf_part(o, i));
                        }
                });
            };
            constexpr std::integral_constant<int, 0> lower;
            constexpr std::integral_constant<int, TH> upper;
            if (ksplit == 1) give(lower);
            __syncthreads();
            if (ksplit == 0) take(lower);
            __syncthreads();
            if (ksplit == 0) give(upper);
            __syncthreads();
            if (ksplit == 1) take(upper);
            __syncthreads();
        }

        // sigma, and in the item's last piece the unquantised tail (one product:
        // T is 0, 8 or 16); this lane's row, 16 tokens per group
        const int ln = lane_now();
        const int fh = ln >> 5, fj = ln & 31;
        const int row = wt * kTile + 32 * (rset & 1) + fj;
        const bool live = wt_raw < a.tiles && row < a.M;
        const float sg = f16(a.sigma[min(row, a.M - 1)]);
        pf_u32x4 bt = {0, 0, 0, 0};
        if (8 * fh < a.T)
            bt = *reinterpret_cast<const pf_u32x4*>(a.codes + a.tail_off +
                                                    2 * (static_cast<size_t>(min(row, a.M - 1)) * a.T + 8 * fh));
        const bool whole = c0 == 0 && c1 == a.upi, tail = a.T > 0 && c1 == a.upi;
        auto load_tail = [&](int t) {
            const uint32_t tok = static_cast<uint32_t>(min(n0 + 32 * (t0 + t) + fj, a.N - 1));
            return __builtin_amdgcn_raw_buffer_load_b128(
                xrs, 8 * fh < a.T ? tok * static_cast<uint32_t>(2 * a.K) + 48u * a.nblk + 16u * fh : 0x80000000u, 0, 0);
        };
        pf_u32x4 at[2] = {};
        if (tail) at[0] = load_tail(0);
        float* slot = nullptr;
        if (S == 2 && !whole)
            slot = a.partials + static_cast<size_t>(2 * blockIdx.x + (u0 >= base ? 0 : 1)) * kPfSlot + 4 * pf_tid();
#pragma unroll
        for (int t = 0; t < TH; ++t) {
            const int tok0 = n0 + 32 * (t0 + t);
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][e] *= sg;
            if (tail) {
                if (t + 1 < TH) at[(t + 1) & 1] = load_tail(t + 1);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, at[t & 1]),
                                                               __builtin_bit_cast(half8_t, bt), acc[t], 0, 0, 0);
            }
            if (S == 2 && t0 + t >= TG) continue;
            if (S == 2 && !whole) {
                // a piece of an item that other workgroups share: slot 0 of the
                // workgroup for the item where its range starts, slot 1 for the
                // item where it ends
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    *reinterpret_cast<pf_u32x4*>(slot + 4 * kPfThreads * (4 * t + k)) =
                        pf_u32x4{pf_bits(acc[t][4 * k]), pf_bits(acc[t][4 * k + 1]), pf_bits(acc[t][4 * k + 2]),
                                 pf_bits(acc[t][4 * k + 3])};
                continue;
            }
            float* yo = a.y + static_cast<size_t>(tok0) * a.M + row;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int tok = 8 * (e >> 2) + 4 * fh + (e & 3);
                if (live && tok0 + tok < a.N) yo[static_cast<size_t>(tok) * a.M] = acc[t][e];
            }
        }
    }
}

// Adds the pieces of the items that several workgroups of gemm_kernel<TG, 2>
// shared, in workgroup order.  A workgroup takes 256 of an item's quads (four
// tokens of a row): quad q of thread t of the product's workgroup.
__global__ __launch_bounds__(256) void gemm_sum_kernel(const GemmArgs a, int tg) {
    const int item = blockIdx.x;
    const unsigned long long base = static_cast<unsigned long long>(item) * a.upi;
    const int wf = pf_worker_of(base, a), wl = pf_worker_of(base + a.upi - 1, a);
    if (wf == wl) return;
    const int at = blockIdx.y * 256 + threadIdx.x;         // quad * 512 + thread of the workgroup
    const int th = (tg + 1) / 2, quad = at / kPfThreads, t = at % kPfThreads;
    const int wave = t >> 6, h = (t >> 5) & 1, j = t & 31;
    const int group = (wave & 1) * th + (quad >> 2);
    const int irow = item / a.tgroups;
    const int row = (irow * 4 + (wave >> 1)) * 32 + j;
    const int tok = (item - irow * a.tgroups) * (32 * tg) + 32 * group + 8 * (quad & 3) + 4 * h;
    if (group >= tg || row >= a.M || tok >= a.N) return;
    const float4* src = reinterpret_cast<const float4*>(a.partials) + at;
    const int side = pf_range_begin(wf, a) >= base ? 0 : 1;
    float4 s = src[static_cast<size_t>(2 * wf + side) * (kPfSlot / 4)];
    for (int w = wf + 1; w <= wl; w += 4) {
        float4 p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) p[u] = src[static_cast<size_t>(2 * min(w + u, wl)) * (kPfSlot / 4)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (w + u <= wl) {
                s.x += p[u].x;
                s.y += p[u].y;
                s.z += p[u].z;
                s.w += p[u].w;
            }
    }
    float* yo = a.y + static_cast<size_t>(tok) * a.M + row;
    yo[0] = s.x;
    if (tok + 1 < a.N) yo[static_cast<size_t>(a.M)] = s.y;
    if (tok + 2 < a.N) yo[2 * static_cast<size_t>(a.M)] = s.z;
    if (tok + 3 < a.N) yo[3 * static_cast<size_t>(a.M)] = s.w;
}

}  // namespace tetra_dev
