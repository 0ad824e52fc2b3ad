// Nearest-point encoder of 24-weight blocks (the offline step of Sec. 3.1,
// run here on the GPU).  Included by tetra.hip after kernels.h.
//
// Shape-gain (Eq. 2): a block comes back as y / ||y|| * gain[g] * sigma, so
// the encoder wants the kept lattice point closest in direction to the
// block.  At each of two trial radii a it takes the kept point nearest to
// a w / ||w||, then keeps the trial point of better direction and the gain
// nearest to the block's projection on it.
//
// Nearest point at one radius.  With integer targets T_j = rint(w_j a 2^16 /
// ||w||) the point maximises S(y) = sum_j (2 T_j y_j - 2^16 y_j^2), an exact
// integer that splits over the three sections of Sec. 3.2.  A section's best
// score is wanted for each parity p, pattern byte P (one of the 128
// even-weight bytes) and class c over the section's list of that class
// (Sec. 3.3: the class halves of the table for sections 1 and 3, the middle
// list for section 2).
//
// The lists need not be scanned for that.  A row's cost is 8 + 8 k with
// k = sum_j t(rank_j), t(r) = r (r + 1) / 2, and its class is k mod 2; a list
// holds every rank vector of its class below its last cost level K, and of
// level K those whose packed row is at most the list's last row.  So:
//   * a quad profile: for each half of the section (coordinates 0-3 or 4-7),
//     p and 4 pattern bits (2 x 2 x 16 = 64 lanes of a wave), the best score
//     of four ranks at every k <= 11, from the profiles of its two pairs;
//   * for the high half also the profile of the quads whose packed ranks H
//     are below the last row's (level K takes any low quad with those), and
//     the one quad H equal to it (level K then takes low quads up to the last
//     row's: one more number per low quad);
//   * a (p, P, c) best is a maximum of about K sums of one low and one high
//     entry.
// About 800 wave instructions replace the scan of 2,048 rows for 256 (p, P)
// pairs.
//
// The join takes the best of the prefix pair (b1) per state s8 and of the
// suffix pair (b3) per state s16 first, then 64 states x 16 branches x p, r,
// delta with r3 = p xor r xor delta (Eq. 3).  Equal sums go to the smallest
// key (s8 | p << 6 | r << 7 | b1 << 8 | b2 << 9 | b3 << 13) * 2 + delta: b1
// and b3 are 0 wherever they reach the same score, and the lanes that hold
// the best sum go over their candidates a second time for the key.  Only
// then are rows looked up: in each section the first row of the winner's list
// that reaches its score, from the start of the lowest level that does.
//
// Work: a workgroup of six waves takes a block at a time, a wave per section
// and radius, and a batch of up to kEncBatch blocks at once for what is one
// lane's work per block (norm, direction, gain: float64 sums in coordinate
// order, the same operations in the same order as any other implementation
// of this definition).  Bound by VALU issue (1,130 instructions per wave, that is
// per section and radius: 0.22 ms of issue for 20,000 blocks): 20,000 Gaussian
// blocks in 0.31 ms, against 26.8 ms for a kernel that scored every row of the
// lists for every (p, P).  Six waves per SIMD (80 registers, eleven of them
// spilled outside the quad profiles) measured 0.33 ms where five without
// spills took 0.37.
#pragma once

namespace tetra_dev {

constexpr int kEncScale = 1 << 16;
constexpr double kEncMaxRadius = 25.0;              // keeps every score inside int32 and 2 T inside 24 bits
constexpr int kEncWaves = 6;                        // section + 3 * trial
constexpr int kEncThreads = 64 * kEncWaves;
constexpr int kEncBatch = 24;                       // blocks whose norms and words are formed together
constexpr int kEncGroupsPerCU = 4;                  // 4 x 40 KB of LDS, 6 waves per SIMD
// Factor that marks a block whose squared norm is zero or not finite (it gets
// the word 0): below every factor of another block, which may be 0 for one
// radius and not for the other
constexpr double kEncZeroBlock = -1.0;

struct EncodeArgs {
    const float* w;                                 // [n][24], block order
    const float* sigma;                             // [n]
    uint16_t* words;                                // [n][3], canonical little-endian
    size_t n;
    double alpha[2];                                // trial radii
};

// value of rank rk in o + 4Z counted outward from zero, positive first at
// equal magnitude (o = p + 2c)
__device__ __forceinline__ int enc_value(int o, int rk) {
    const int p = o & 1, c = o >> 1;
    const int u = 2 * rk + 1;
    const int neg = (rk ^ c ^ p ^ 1) & 1;
    return (neg ? -u : u) + (1 - p);
}

// 2 T v - 2^16 v^2 (|2 T - 2^16 v| < 2^22: a 24-bit multiply)
__device__ __forceinline__ int enc_score(int t2, int v) { return __mul24(v, t2 - (v << 16)); }

// ---- the lists' last rows: cost level and ranks (checked by the table generator)

constexpr int enc_t(int r) { return r * (r + 1) / 2; }
constexpr int kEncRanks = 5;                        // ranks 0..4: t(5) exceeds every K
constexpr int kEncLevels = 12;                      // k = 0..11

struct EncLast {
    uint32_t row;
    constexpr int rank(int j) const { return static_cast<int>(row >> (4 * j) & 15u); }
    constexpr int level(int j0, int j1) const {
        int k = 0;
        for (int j = j0; j < j1; ++j) k += enc_t(rank(j));
        return k;
    }
    constexpr int K() const { return level(0, 8); }
};

constexpr EncLast enc_last(bool middle, int c) {
    return EncLast{middle ? (c ? tetra::kMidLastRow1 : tetra::kMidLastRow0)
                          : (c ? tetra::kLastRow1 : tetra::kLastRow0)};
}
static_assert(enc_last(false, 0).K() < kEncLevels && enc_last(false, 1).K() < kEncLevels &&
                  enc_last(true, 0).K() < kEncLevels && enc_last(true, 1).K() < kEncLevels,
              "levels of the quad profiles");
static_assert(enc_last(false, 0).K() % 2 == 0 && enc_last(false, 1).K() % 2 == 1 &&
                  enc_last(true, 0).K() % 2 == 0 && enc_last(true, 1).K() % 2 == 1,
              "class = level mod 2");

// Inside a section a score S of level k is kept as 16 S - k: the best of a
// set is then the best score and, of equal scores, the lowest level, where
// the first row of the list lies.  A quad of level <= 11 has |y|^2 <= 136 and
// so -2^16 (50 * 11.7 + 136) <= S <= 2^16 * 625 at the largest radius: 16 S
// stays above -2^29.5 and below 2^29.3, sums of two inside int32.  kEncNone
// stands for no quad: with any other entry it stays below every section's
// best, which is at least that of the row of ranks 0 or of a row with one
// rank 1 (|y|^2 <= 32: 16 S > -2^28.3, against -2^30 + 2^29.3).
constexpr int kEncNone = -(1 << 30);
constexpr int kEncUnit = 16;

__device__ __forceinline__ int enc_tagged_score(int tag) { return (tag + kEncUnit - 1) >> 4; }
__device__ __forceinline__ int enc_tagged_level(int tag) { return -tag & (kEncUnit - 1); }

// first row of level k in the list of class k mod 2 (checked by the table generator)
__device__ const uint16_t g_enc_level_row[kEncLevels] = TETRA_LEVEL_ROWS;

// best score per level of some ranks; levels no rank vector has are unset,
// which is known when the loops below are unrolled
struct EncProfile {
    int s[kEncLevels];
    bool has[kEncLevels];
    __device__ __forceinline__ EncProfile() {
#pragma unroll
        for (int k = 0; k < kEncLevels; ++k) {
            s[k] = kEncNone;
            has[k] = false;
        }
    }
    __device__ __forceinline__ void put(int k, int v) {
        s[k] = has[k] ? max(s[k], v) : v;
        has[k] = true;
    }
};

typedef int enc_i2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ enc_i2 enc_pair(int x, int y) { return enc_i2{x, y}; }

// orders a wave's LDS accesses before and after it (all lanes of one wave)
__device__ __forceinline__ void enc_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

typedef int EncE[4][kEncRanks];                     // scores of a quad's coordinates by rank

// pairs (ranks of coordinates j, j + 1 of the quad) whose packed value is
// below (Below) rank pair (ra, rb), or every pair
template <bool Below>
__device__ __forceinline__ EncProfile enc_pairs(const EncE& e, int j, int ra, int rb, bool equal, int most) {
    EncProfile f;
#pragma unroll
    for (int b = 0; b < kEncRanks; ++b)
#pragma unroll
        for (int a = 0; a < kEncRanks; ++a) {
            const int k = enc_t(a) + enc_t(b);
            if (k > most) continue;
            if (Below && !(b < rb || (b == rb && (equal ? a <= ra : a < ra)))) continue;
            f.put(k, e[j][a] + e[j + 1][b]);
        }
    return f;
}

// adds to f the quads made of a pair of lo and a pair of hi, up to level K
__device__ __forceinline__ void enc_join(EncProfile& f, const EncProfile& lo, const EncProfile& hi, int K) {
#pragma unroll
    for (int a = 0; a < kEncLevels; ++a)
#pragma unroll
        for (int b = 0; b < kEncLevels; ++b)
            if (a + b <= K && lo.has[a] && hi.has[b]) f.put(a + b, lo.s[a] + hi.s[b]);
}

// LDS of a wave: the low quads' entries (12 levels, then one number per
// class), the high quads' entries (12 levels per class, then one number per
// class), strides that spread 16 of them over all banks.  The section's
// results then take the place of the low quads.
constexpr int kEncLoStride = 20, kEncHiStride = 28;
constexpr int kEncWaveWords = 32 * (kEncLoStride + kEncHiStride);
constexpr int kEncPickOff = 32 * kEncLoStride;      // scores of the winner's coordinates by rank: [8][8]

// The wave's quad profiles into its LDS: lane = h << 5 | p << 4 | pattern
// bits of coordinates 4h..4h+3, t2[j] = 2 T of those coordinates.
template <bool Middle>
__device__ __forceinline__ void enc_profiles(int* W, int lane, const int (&t2)[4]) {
    const int most = enc_last(Middle, 0).K() > enc_last(Middle, 1).K() ? enc_last(Middle, 0).K() : enc_last(Middle, 1).K();
    EncE e;
    {
        // 16 (2 T v - 2^16 v^2) - t(r) = V (2 T - 2^12 V) - t(r) with V = 16 v =
        // +-16 (2 r + 1) + 16 (1 - p), the sign alternating with r: three 24-bit multiply-adds (the factors are kept opaque:
        // the compiler would form them by selects and shifts)
        const int q16 = ~lane & 16;
        int m = -4096;
        asm("" : "+s"(m));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int s16 = ((lane >> j) ^ (lane >> 4)) & 1 ? 16 : -16;     // c xor p
            asm("" : "+v"(s16));
#pragma unroll
            for (int r = 0; r < kEncRanks; ++r) {
                int V = __mul24(s16, r & 1 ? -(2 * r + 1) : 2 * r + 1) + q16;
                asm("" : "+v"(V));
                int x = __mul24(V, m) + t2[j];
                asm("" : "+v"(x));
                e[j][r] = __mul24(V, x) - enc_t(r);
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    const EncProfile lo = enc_pairs<false>(e, 0, 0, 0, false, most);
    EncProfile all;
    {
        const EncProfile hi = enc_pairs<false>(e, 2, 0, 0, false, most);
        enc_join(all, lo, hi, most);
    }
    __builtin_amdgcn_sched_barrier(0);
    int* const low = W + (lane & 31) * kEncLoStride;
    int* const high = W + 32 * kEncLoStride + (lane & 31) * kEncHiStride;
    const bool is_low = lane < 32;
    if (is_low) {
#pragma unroll
        for (int k = 0; k <= most; ++k) low[k] = all.s[k];
    }
    // as a high quad: any quad two or more levels below (through LDS rather
    // than registers to the maximum with the level's own quads)
    if (!is_low) {
#pragma unroll
        for (int k = 2; k <= most; ++k) all.s[k] = max(all.s[k], all.s[k - 2]);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k <= enc_last(Middle, c).K(); ++k) high[kEncLevels * c + k] = k < 2 ? kEncNone : all.s[k - 2];
    }
    enc_wave_sync();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        // one class's registers at a time, the sums of pairs formed anew (kept
        // from above they would be spilled)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < kEncRanks; ++r) asm volatile("" : "+v"(e[j][r]));
        __builtin_amdgcn_sched_barrier(0);
        const EncLast last = enc_last(Middle, c);
        const int K = last.K();
        // as a high quad: level K takes the quads packed below the last row's
        EncProfile cut;
        {
            const EncProfile hb = enc_pairs<true>(e, 2, last.rank(6), last.rank(7), false, K);
            enc_join(cut, lo, hb, K);
            __builtin_amdgcn_sched_barrier(0);
            const EncProfile lb = enc_pairs<true>(e, 0, last.rank(4), last.rank(5), false, K);
            const int k67 = last.level(6, 8), s67 = e[2][last.rank(6)] + e[3][last.rank(7)];
#pragma unroll
            for (int k = 0; k < kEncLevels; ++k)
                if (lb.has[k] && k + k67 <= K) cut.put(k + k67, lb.s[k] + s67);
        }
        __builtin_amdgcn_sched_barrier(0);
        const int eq_high = e[0][last.rank(4)] + e[1][last.rank(5)] + e[2][last.rank(6)] + e[3][last.rank(7)];
        // as a low quad beside the last row's own high quad: level K exactly,
        // packed up to the last row's
        const int kl = last.level(0, 4), k23 = last.level(2, 4);
        EncProfile eq;
        {
            const EncProfile hb = enc_pairs<true>(e, 2, last.rank(2), last.rank(3), false, K);
#pragma unroll
            for (int a = 0; a < kEncLevels; ++a)
#pragma unroll
                for (int b = 0; b < kEncLevels; ++b)
                    if (a + b == kl && lo.has[a] && hb.has[b]) eq.put(kl, lo.s[a] + hb.s[b]);
            const EncProfile lb = enc_pairs<true>(e, 0, last.rank(0), last.rank(1), true, K);
            if (lb.has[kl - k23]) eq.put(kl, lb.s[kl - k23] + e[2][last.rank(2)] + e[3][last.rank(3)]);
        }
        if (is_low) {
            low[kEncLevels + c] = eq.s[kl];
        } else {
#pragma unroll
            for (int k = 0; k <= K; ++k) {
                if (cut.has[k]) high[kEncLevels * c + k] = max(high[kEncLevels * c + k], cut.s[k]);
            }
            high[2 * kEncLevels + c] = eq_high;
        }
    }
}

// best score of class c (0, 1) of the section for parity p and pattern byte P
template <bool Middle>
__device__ __forceinline__ void enc_best(const int* W, int p, uint32_t P, int (&best)[2]) {
    const int* const low = W + (16 * p + (P & 15)) * kEncLoStride;
    const int* const high = W + 32 * kEncLoStride + (16 * p + (P >> 4)) * kEncHiStride;
    int l[kEncLevels];
#pragma unroll
    for (int k = 0; k < kEncLevels; ++k) l[k] = low[k];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int K = enc_last(Middle, c).K();
        int b = low[kEncLevels + c] + high[2 * kEncLevels + c];
#pragma unroll
        for (int k = 0; k <= K; ++k) b = max(b, l[k] + high[kEncLevels * c + K - k]);
        best[c] = b;
    }
}

// pattern byte b of pair s: the 64 pairs {P, ~P} in order of their smaller
// byte, which has bit 7 clear and even weight, hence (s << 1) | parity(s)
__device__ __forceinline__ uint32_t enc_byte(int s, int b) {
    const uint32_t rep = static_cast<uint32_t>(s) << 1 | (__builtin_popcount(s) & 1);
    return b ? rep ^ 255u : rep;
}

// Results of a section's wave, over its low-quad entries:
//   sections 1, 3: [p][s][c] best score of the pair s; the bytes at
//     kEncBitOff hold per (p, s) the bits c that only the pair's second byte
//     reaches;
//   section 2: [p][P & 127][c];
//   the bytes at kEncLevelOff hold the levels of these bests, class 0 in the
//   low four bits: [p][s][b], in section 2 [p][P & 127].
constexpr int kEncBitOff = 512, kEncLevelOff = kEncBitOff + 32;
static_assert(kEncBatch <= 64, "a lane per block");
static_assert(kEncLevelOff + 64 <= kEncPickOff, "results fit over the low quads");

template <bool Middle>
__device__ __forceinline__ void enc_section(int* W, int lane, const int (&t2)[4]) {
    enc_profiles<Middle>(W, lane, t2);
    enc_wave_sync();
    int best[2][2][2];                              // [p][b][c]
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            enc_best<Middle>(W, p, enc_byte(lane, b), best[p][b]);
            __builtin_amdgcn_sched_barrier(0);
        }
    enc_wave_sync();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        uint8_t level[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            level[b] = static_cast<uint8_t>(enc_tagged_level(best[p][b][0]) | enc_tagged_level(best[p][b][1]) << 4);
#pragma unroll
            for (int c = 0; c < 2; ++c) best[p][b][c] = enc_tagged_score(best[p][b][c]);
        }
        if (Middle) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const uint32_t i7 = enc_byte(lane, b) & 127u;
                *reinterpret_cast<enc_i2*>(W + 256 * p + 2 * i7) = enc_pair(best[p][b][0], best[p][b][1]);
                reinterpret_cast<uint8_t*>(W + kEncLevelOff)[128 * p + i7] = level[b];
            }
        } else {
            reinterpret_cast<uint16_t*>(W + kEncLevelOff)[64 * p + lane] = static_cast<uint16_t>(level[0] | level[1] << 8);
            *reinterpret_cast<enc_i2*>(W + 128 * p + 2 * lane) =
                enc_pair(max(best[p][0][0], best[p][1][0]), max(best[p][0][1], best[p][1][1]));
            reinterpret_cast<uint8_t*>(W + kEncBitOff)[64 * p + lane] = static_cast<uint8_t>(
                (best[p][1][0] > best[p][0][0] ? 1 : 0) | (best[p][1][1] > best[p][0][1] ? 2 : 0));
        }
    }
}

// key bits of a winner
struct EncKey {
    int d, s8, p, r, b1, b2, b3;
    __device__ __forceinline__ explicit EncKey(int k)
        : d(k & 1), s8((k >> 1) & 63), p((k >> 7) & 1), r((k >> 8) & 1), b1((k >> 9) & 1), b2((k >> 10) & 15),
          b3((k >> 14) & 1) {}
    // class of a section's row and its pattern byte; path: path_bytes entry of (s8, b2)
    __device__ __forceinline__ int cls(int sec) const { return sec == 0 ? r : sec == 1 ? d : p ^ r ^ d; }
    __device__ __forceinline__ uint32_t byte(int sec, uint32_t path) const {
        return sec == 0 ? enc_byte(s8, b1) : sec == 1 ? (path >> 8) & 255u : ((path >> 16) & 255u) ^ (b3 ? 255u : 0u);
    }
};

// b2 of branch i of the join's wave `sec` of three: sec + 3 i (of the waves
// with five, the sixth repeats the fifth)
__device__ __forceinline__ int enc_b2(int sec, int i) { return sec + 3 * i > 15 ? sec + 3 * (i - 1) : sec + 3 * i; }

// smallest key of the sums of state s8, parity p and a branch that equal top
__device__ __forceinline__ int enc_smallest_key(const int* W1, const int* W2, const int* W3, int s8, int p,
                                                uint32_t path, int b2, int top) {
    const int s16 = path >> 17;
    const enc_i2 A = *reinterpret_cast<const enc_i2*>(W1 + 128 * p + 2 * s8);
    const enc_i2 B = *reinterpret_cast<const enc_i2*>(W2 + 256 * p + 2 * ((path >> 8) & 127u));
    const enc_i2 C = *reinterpret_cast<const enc_i2*>(W3 + 128 * p + 2 * s16);
    const int ab = reinterpret_cast<const uint8_t*>(W1 + kEncBitOff)[64 * p + s8];
    const int cb = reinterpret_cast<const uint8_t*>(W3 + kEncBitOff)[64 * p + s16];
    int best = INT_MAX;
#pragma unroll
    for (int rd = 0; rd < 4; ++rd) {
        const int r = rd >> 1, d = rd & 1, r3 = p ^ r ^ d;
        const int sum = (r ? A.y : A.x) + (d ? B.y : B.x) + (r3 ? C.y : C.x);
        const int key = d | s8 << 1 | p << 7 | r << 8 | ((ab >> r) & 1) << 9 | b2 << 10 | ((cb >> r3) & 1) << 14;
        if (sum == top) best = min(best, key);
    }
    return best;
}

__global__ __launch_bounds__(kEncThreads) __attribute__((amdgpu_waves_per_eu(6, 6))) void encode_kernel(const EncodeArgs a) {
    __shared__ __attribute__((aligned(16))) int s_wave[kEncWaves][kEncWaveWords];
    __shared__ float s_w[kEncBatch * 24];
    __shared__ double s_f[2][kEncBatch];            // radius 2^16 / ||w|| (0 where it underflows), or kEncZeroBlock for both
    __shared__ int s_score[kEncWaves], s_key[kEncWaves];   // a wave's best sum of the join and its key
    __shared__ int s_pick[kEncBatch][2][4];         // per trial: key, rows of the three sections
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int trial = wave >= 3 ? 1 : 0, sec = wave - 3 * trial;
    int* const W = s_wave[wave];
    const int* const W1 = s_wave[3 * trial], * const W2 = s_wave[3 * trial + 1], * const W3 = s_wave[3 * trial + 2];
    // the join's branches of this wave: b2 = sec, sec + 3, ..; lane = s8
    uint32_t branches[3];                           // two each: P2 & 127 | s16 << 8
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        branches[i] = 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t path = g_canonical.path_bytes[enc_b2(sec, 2 * i + u) << 7 | (threadIdx.x & 63)];
            branches[i] |= (((path >> 8) & 127u) | (path >> 17) << 8) << (16 * u);
        }
    }
    // contiguous blocks per workgroup, in batches
    const size_t first = pf_uniform(a.n * blockIdx.x / gridDim.x), end = pf_uniform(a.n * (blockIdx.x + 1) / gridDim.x);
    for (size_t b0 = first; b0 < end; b0 += kEncBatch) {
        const int nb = static_cast<int>(end - b0 < kEncBatch ? end - b0 : kEncBatch);
        __syncthreads();                            // the previous batch's words are formed
        for (int i = 64 * wave + lane_now(); i < 24 * nb; i += kEncThreads) s_w[i] = a.w[24 * b0 + i];
        __syncthreads();
        if (wave == 0 && lane_now() < nb) {
            const int blk = lane_now();
            const float* w = s_w + 24 * blk;
            double n2 = 0.0;
            for (int j = 0; j < 24; ++j) n2 += static_cast<double>(w[j]) * static_cast<double>(w[j]);
            const bool zero = !(n2 > 0.0) || !(n2 <= 1.0e300);
            const double rn = zero ? 1.0 : sqrt(n2);
#pragma unroll
            for (int q = 0; q < 2; ++q) s_f[q][blk] = zero ? kEncZeroBlock : a.alpha[q] * static_cast<double>(kEncScale) / rn;
        }
        __syncthreads();
        for (int blk = 0; blk < nb; ++blk) {
            const double f = s_f[trial][blk];
            if (f == kEncZeroBlock) continue;       // of both radii: every wave leaves out the barriers below, or none
            // read afresh for each block: what derives from the lane alone would
            // otherwise be kept in registers across the blocks, and spilled
            const int lane = lane_now();
            {
                int t2[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    t2[j] = 2 * static_cast<int>(rint(static_cast<double>(s_w[24 * blk + 8 * sec + 4 * (lane >> 5) + j]) * f));
                if (sec == 1)
                    enc_section<true>(W, lane, t2);
                else
                    enc_section<false>(W, lane, t2);
            }
            __syncthreads();
            // join: the best sum of this wave's branches, then its smallest key
            int sum[2][6], js = INT_MIN;
            uint32_t branch[6];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                asm volatile("" : "+v"(branches[i]));   // no address of it kept across the blocks
                branch[2 * i] = branches[i] & 0xFFFFu;
                branch[2 * i + 1] = branches[i] >> 16;
            }
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const enc_i2 A = *reinterpret_cast<const enc_i2*>(W1 + 128 * p + 2 * lane);
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    const enc_i2 B = *reinterpret_cast<const enc_i2*>(W2 + 256 * p + 2 * (branch[i] & 127u));
                    const enc_i2 C = *reinterpret_cast<const enc_i2*>(W3 + 128 * p + 2 * (branch[i] >> 8));
                    // r xor delta = 0, then 1
                    sum[p][i] = max(max(A.x + B.x, A.y + B.y) + (p ? C.y : C.x), max(A.x + B.y, A.y + B.x) + (p ? C.x : C.y));
                    js = max(js, sum[p][i]);
                }
            }
            int top = js;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) top = max(top, __shfl_xor(top, off, 64));
            int jk = INT_MAX;
            uint32_t hits = 0;
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int i = 0; i < 6; ++i) hits |= sum[p][i] == top ? 1u << (6 * p + i) : 0u;
            while (hits) {
                const int it = __builtin_ctz(hits), p = it >= 6, b2 = enc_b2(sec, it - 6 * p);
                hits &= hits - 1;
                const uint32_t path = g_canonical.path_bytes[b2 << 7 | lane];
                jk = min(jk, enc_smallest_key(W1, W2, W3, lane, p, path, b2, top));
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) jk = min(jk, __shfl_xor(jk, off, 64));
            if (lane == 0) {
                s_score[wave] = top;
                s_key[wave] = jk;
            }
            __syncthreads();
            // the trial's point: each section's wave finds its row
            int ws = s_score[3 * trial], wk = s_key[3 * trial];
#pragma unroll
            for (int q = 1; q < 3; ++q) {
                const int os = s_score[3 * trial + q], ok = s_key[3 * trial + q];
                if (os > ws || (os == ws && ok < wk)) {
                    ws = os;
                    wk = ok;
                }
            }
            wk = __builtin_amdgcn_readfirstlane(wk);
            const EncKey key(wk);
            const uint32_t P = key.byte(sec, g_canonical.path_bytes[key.s8 | key.b2 << 7]);
            const int cls = key.cls(sec);
            // the score it has and the level its row lies in
            const int s16 = static_cast<int>((P & 128u ? ~P : P) & 127u) >> 1;
            const int want = sec == 1 ? W[256 * key.p + 2 * static_cast<int>(P & 127u) + cls]
                                      : W[128 * key.p + 2 * s16 + cls];
            const int levels = reinterpret_cast<const uint8_t*>(
                W + kEncLevelOff)[128 * key.p + (sec == 1 ? static_cast<int>(P & 127u) : 2 * s16 + static_cast<int>(P >> 7))];
            const int start = __builtin_amdgcn_readfirstlane(g_enc_level_row[(levels >> (4 * cls)) & 15]);
            {
                // scores of the section's coordinates by rank (j = lane / 8)
                const int j = lane >> 3, o = key.p + 2 * static_cast<int>((P >> j) & 1u);
                const int t2 = 2 * static_cast<int>(rint(static_cast<double>(s_w[24 * blk + 8 * sec + j]) * f));
                W[kEncPickOff + lane] = enc_score(t2, enc_value(o, lane & 7));
            }
            enc_wave_sync();
            const uint32_t* const rows = g_canonical.rows + 2048 * cls;
            int at = start;
            uint32_t row[2] = {rows[min(start + lane, 2047)], rows[min(start + 64 + lane, 2047)]};
            for (int i = start; i < 2048; i += 128) {
                const uint32_t next[2] = {rows[min(i + 128 + lane, 2047)], rows[min(i + 192 + lane, 2047)]};
                unsigned long long hit[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    int sc = 0;
#pragma unroll
                    for (int j = 0; j < 8; ++j) sc += W[kEncPickOff + 8 * j + static_cast<int>((row[u] >> (4 * j)) & 7u)];
                    hit[u] = __ballot(sc == want);
                }
                if (hit[0] | hit[1]) {
                    at = i + (hit[0] ? __builtin_ctzll(hit[0]) : 64 + __builtin_ctzll(hit[1]));
                    break;
                }
                row[0] = next[0];
                row[1] = next[1];
            }
            if (lane == 0) {
                s_pick[blk][trial][1 + sec] = at;
                if (sec == 0) s_pick[blk][trial][0] = wk;
            }
        }
        __syncthreads();
        // a lane per block: the trial of better direction, the gain, the word
        if (wave == 0 && lane_now() < nb) {
            const int blk = lane_now();
            const size_t gb = b0 + blk;
            uint64_t word = 0;
            if (s_f[0][blk] != kEncZeroBlock) {
                double best_c = 0.0;
                int best_t = 0;
#pragma unroll 1
                for (int tr = 0; tr < 2; ++tr) {
                    const EncKey key(s_pick[blk][tr][0]);
                    const uint32_t path = g_canonical.path_bytes[key.s8 | key.b2 << 7];
                    double dot = 0.0, yy = 0.0;
#pragma unroll 1
                    for (int s = 0; s < 3; ++s) {
                        const uint32_t P = key.byte(s, path);
                        const uint32_t rho = g_canonical.rows[key.cls(s) << 11 | s_pick[blk][tr][1 + s]];
                        for (int q = 0; q < 8; ++q) {
                            const int o = key.p + 2 * static_cast<int>((P >> q) & 1u);
                            const int v = enc_value(o, static_cast<int>((rho >> (4 * q)) & 15u));
                            dot += static_cast<double>(s_w[24 * blk + 8 * s + q]) * static_cast<double>(v);
                            yy += static_cast<double>(v) * static_cast<double>(v);
                        }
                    }
                    const double ny = sqrt(yy);
                    const double cdir = ny > 0.0 ? dot / ny : -INFINITY;
                    if (tr == 0 || cdir > best_c) {
                        best_c = cdir;
                        best_t = tr;
                    }
                }
                // the gain nearest to the projection, then the canonical word
                const double gs = static_cast<double>(a.sigma[gb]);
                const double d0 = static_cast<double>(g_canonical.gain[0]) * gs - best_c;
                const double d1 = static_cast<double>(g_canonical.gain[1]) * gs - best_c;
                const uint64_t g = d1 * d1 < d0 * d0 ? 1u : 0u;
                const EncKey k(s_pick[blk][best_t][0]);
                const uint64_t i1 = s_pick[blk][best_t][1];
                const uint64_t i2 = s_pick[blk][best_t][2] + (k.d ? tetra::kMidClass0Rows : 0u);
                const uint64_t i3 = s_pick[blk][best_t][3];
                word = static_cast<uint64_t>(k.s8 | k.p << 6 | k.r << 7 | k.b1 << 8 | k.b2 << 9 | k.b3 << 13) | g << 14 |
                       i1 << 15 | i2 << 26 | i3 << 37;
            }
            uint16_t* out = a.words + 3 * gb;
            out[0] = static_cast<uint16_t>(word);
            out[1] = static_cast<uint16_t>(word >> 16);
            out[2] = static_cast<uint16_t>(word >> 32);
        }
    }
}

}  // namespace tetra_dev
