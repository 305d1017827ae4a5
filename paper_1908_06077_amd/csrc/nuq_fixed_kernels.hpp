// Fixed-width coding (Sec. 5: the "4-bit" and "8-bit" variants; 3 bits in Table 1): every coordinate sends its sign
// and level index in b bits.  Layout: coordinate i of a bucket is the code  sign << (b-1) | level index  at bits
// [i*b, i*b + b) of the bucket's field, most significant bit first, in 32-bit words; every bucket's field is
// wpb = ceil(bucket * b / 32) words, so bucket k starts at word k * wpb.  No offsets, no index: both directions are
// plain streaming kernels.
#pragma once

#include "nuq_encode_kernels.hpp"

namespace nuq {

struct FixedParams {
    uint32_t b;     // bits per coordinate, 3..8
    uint32_t wpb;   // words per bucket field
};

// LDS words per team of k_pack_fixed: [qb32: rows * TEAM][field: wpb][scratch: 64]
__host__ __device__ inline uint32_t fixed_lds_words(uint32_t rows, uint32_t team, uint32_t wpb)
{
    const uint32_t w = (rows * team + wpb + 1u) & ~1u;
    return w + 64u;
}

// MODE 0: norms + quantizer + packing from v (read once).  MODE 1: packing of level|sign bytes.  MODE 2: as 0 for the
// level table T and the norm P.norm_linf selects (T is ignored in the other modes).  One bucket per team.
template <int TEAM, int VPT, int MODE>
__global__ __launch_bounds__(TeamGeom<TEAM>::kWG) void k_pack_fixed(EncodeParams P, EncodeBatch Wk, FixedParams F,
                                                                    LevelTable T)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const EncodeWorker &W = Wk.w[blockIdx.y];
    const uint32_t tid = threadIdx.x % TEAM;
    const uint32_t team = team_uniform_u32<TEAM>(threadIdx.x / TEAM);
    uint32_t *lds = smem + team * P.lds_words;
    uint32_t *qb32 = lds;
    uint32_t *field = qb32 + P.rows * TEAM;
    uint32_t *scratch = lds + P.lds_words - 64u;
    const uint64_t b = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG + team;
    const bool active = b < P.nb;
    const uint64_t base = active ? b * P.bucket : 0;
    const uint32_t nbk = active ? (uint32_t)min((uint64_t)P.bucket, P.d - base) : 0u;

    for (uint32_t i = tid; i < F.wpb; i += TEAM)
        field[i] = 0u;
    if constexpr (MODE == 2)
        front_quantize_table_to_lds<TEAM, VPT>(P, W, T, b, active, base, nbk, tid, qb32, scratch, PlainBytes{}, [] {});
    else if constexpr (MODE == 0)
        front_quantize_to_lds<TEAM, VPT>(P, W, b, active, base, nbk, tid, qb32, scratch, PlainBytes{}, [] {});
    else
        front_bytes_to_lds<TEAM, VPT>(P, W, base, nbk, tid, qb32);
    __syncthreads();

    // Each thread packs a contiguous chunk of rows * 4 coordinates.  Codes are shifted into a 64-bit register and
    // leave it 32 bits at a time; a chunk's first and last words may be shared with its neighbours, so words are
    // OR-ed into the (zeroed) field.
    const uint32_t per = P.rows * 4u;
    const uint32_t c0 = tid * per;
    const uint32_t c1 = min(c0 + per, nbk);
    if (c0 < c1) {
        const uint8_t *qbytes = reinterpret_cast<const uint8_t *>(qb32);
        const uint32_t bit0 = c0 * F.b;
        uint32_t wi = bit0 >> 5, fill = bit0 & 31u;
        uint64_t acc = 0;
        for (uint32_t c = c0; c < c1; ++c) {
            const uint32_t byte = qbytes[c];
            const uint32_t code = ((byte >> 7) << (F.b - 1u)) | (byte & 0x7fu);
            acc = (acc << F.b) | code;
            fill += F.b;
            if (fill >= 32u) {
                fill -= 32u;
                atomicOr(&field[wi++], (uint32_t)(acc >> fill));
                acc &= (1ull << fill) - 1ull;
            }
        }
        if (fill)
            atomicOr(&field[wi], (uint32_t)(acc << (32u - fill)));
    }
    team_barrier<TEAM>();
    if (active) {
        uint32_t *dst = W.words + b * F.wpb;
        for (uint32_t i = tid; i < F.wpb; i += TEAM)
            dst[i] = field[i];
    }
}

// ---- 4 and 8 bits: no LDS phase ----------------------------------------------------------------------------------
// At these widths the four coordinates that a thread holds of a row are a whole piece of the field: at 8 bits its word,
// at 4 bits half a word whose other half is its neighbour's.  So the codes go from registers to memory: 4 bytes per lane
// and row, whole 256-byte runs per wave (at 4 bits two rows share an instruction: even lanes store their pair's word of
// the first row, odd lanes that of the second).  Through LDS (k_pack_fixed: bytes out, contiguous chunks in, field OR-ed
// together, field out, two barriers) the same codes cost 8 instructions per coordinate more.  Eight gradients of 25.6 M
// coordinates at 4 bits: QSGDinf (bound by vector issue) 269 -> 226 us with the unpack; the main scheme's pack stays at
// 147 us = 6.3 TB/s, what a bare kernel that reads as much and writes an eighth of it reaches.

// The four level|sign bytes of a word as four 4-bit codes (sign << 3 | level), the first on top.  A level above 7 is the
// caller's error; its bit 3 meets the sign's, so that 8 is the signed zero that a receiver refuses, as at the other widths.
__device__ __forceinline__ uint32_t nibble_codes(uint32_t bytes)
{
    const uint32_t n = ((bytes >> 4) & 0x08080808u) | (bytes & 0x0f0f0f0fu);
    const uint32_t hi = __builtin_amdgcn_udot4(n, 0x00000110u, 0u, false);      // n0 << 4 | n1
    return __builtin_amdgcn_udot4(n, 0x01100000u, hi << 8, false);              // ... | n2 << 4 | n3
}

// MODE as k_pack_fixed; B = 4 or 8.
template <int TEAM, int VPT, int MODE, int B>
__global__ __launch_bounds__(TeamGeom<TEAM>::kWG) void k_pack_fixed_direct(EncodeParams P, EncodeBatch Wk, FixedParams F,
                                                                           LevelTable T)
{
    static_assert(B == 4 || B == 8, "codes of a thread's row must be whole halfwords");
    __shared__ __align__(8) uint32_t scratch_all[TeamGeom<TEAM>::kTeamsPerWG][64];
    __shared__ uint32_t part[TEAM > kWave ? kNormParts<TEAM> * TEAM : 1];
    const EncodeWorker &W = Wk.w[blockIdx.y];
    const uint32_t tid = threadIdx.x % TEAM;
    const uint32_t team = team_uniform_u32<TEAM>(threadIdx.x / TEAM);
    uint32_t *scratch = scratch_all[team];
    const uint64_t b = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG + team;
    const bool active = b < P.nb;
    const uint64_t base = active ? b * P.bucket : 0;
    const uint32_t nbk = active ? (uint32_t)min((uint64_t)P.bucket, P.d - base) : 0u;
    uint32_t *const dst = W.words + (active ? b : 0) * F.wpb;
    const uint32_t words = active ? F.wpb : 0u;             // words of the field that exist
    const uint32_t odd = tid & 1u;
    uint32_t codes[B == 4 ? VPT : 1] = {};
    auto put = [&](int i, uint32_t bytes) {
        if constexpr (B == 8) {
            const uint32_t w = (uint32_t)i * TEAM + tid;
            if (w < words)
                dst[w] = __builtin_bswap32(bytes);          // level|sign bytes are the codes; the first one goes on top
        } else {
            codes[i] = nibble_codes(bytes);
        }
    };
    if constexpr (MODE == 2)
        front_quantize_table<TEAM, VPT>(P, W, T, b, active, base, nbk, tid, part, scratch, PlainBytes{}, put, [] {});
    else if constexpr (MODE == 0)
        front_quantize<TEAM, VPT>(P, W, b, active, base, nbk, tid, part, scratch, PlainBytes{}, put, [] {});
    else
        front_bytes<TEAM, VPT>(P, W, base, nbk, tid, put);
    if constexpr (B == 4) {
#pragma unroll
        for (int i = 0; i < VPT; i += 2) {
            if ((uint32_t)i < P.rows) {
                const uint32_t own = codes[i] | (codes[i + 1] << 16);
                const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xf, 0xf, true);   // lane ^ 1
                const uint32_t word = odd ? (other & 0xffff0000u) | (own >> 16) : (own << 16) | (other & 0xffffu);
                const uint32_t w = ((uint32_t)(i + (int)odd) * TEAM + tid) >> 1;
                if (w < words)
                    dst[w] = word;
            }
        }
    }
}

struct UnpackParams {
    const float *norms[kMaxBatch];
    const uint32_t *packed[kMaxBatch];
    float *out;
    uint32_t *flags;
    uint64_t d;
    uint32_t K;
    uint32_t bucket;
    uint32_t s;
    uint32_t b;
    uint32_t wpb;
    uint32_t lut_tabs;          // table variant: buckets a workgroup can touch (tables per worker in LDS)
    float scale;
    int accumulate;
    uint32_t use_levels;        // 1: level j has the value lev[j] (a level table), 0: 2^(j - 1 - s)
    float lev[16];
};

// norm * l_level, exact in fp64 either way (level 1..s+1).
__device__ __forceinline__ double fixed_level_value(const UnpackParams &P, double nrm, uint32_t level)
{
    return P.use_levels ? nrm * (double)P.lev[level] : ldexp(nrm, (int)level - 1 - (int)P.s);
}

// out[i] = [out[i] +] scale * sum_k norms_k[bucket] * sign * 2^(level - 1 - s): fp64 sum in worker order, rounded to
// fp32 (the prior, when there is one, is added in fp32 after that).  A level index above s + 1, or a signed zero,
// raises the malformed flag.
//
// Buckets that are multiples of 32 coordinates: a thread owns 32 consecutive coordinates, i.e. exactly B whole words
// of every worker's field (one contiguous load per worker, coalesced over the wave), and the workgroup's 8192 results
// go through LDS so that the stores are whole lines too.
//
// kLut (3, 5, 6 and 7 bits; at 4 and 8 k_unpack_accumulate_fixed_direct is the variant with tables): the value of every
// code, norm * sign * 2^(level - 1 - s) in fp64 (0 for level 0 and for codes that are not valid), is tabulated in LDS once
// per (bucket the workgroup touches, worker); a code then costs a bit-field extract, an LDS read and an fp64 add instead of
// the exponent arithmetic.  A table of 16 entries is 128 bytes = all 32 banks once, so lanes that read one table never
// conflict whatever their codes.  Codes wider than 5 bits index 32 entries by (sign, low four level bits): levels stop at
// 15.  `lut_tabs` tables per worker are laid out bucket-major.
constexpr uint32_t fixed_lut_entries(uint32_t b) { return b <= 5u ? 1u << b : 32u; }

template <int B>
__device__ __forceinline__ uint32_t fixed_lut_index(uint32_t code)
{
    if constexpr (B <= 5)
        return code;
    else
        return ((code >> (B - 1)) << 4) | (code & 15u);
}

// Whole words of codes that never straddle a word (B = 4, 8): true if some code has a level above s + 1 or is a
// signed zero.  Per field: level + (2^(B-1) - 1) sets the top bit iff level >= 1; level + (2^(B-1) - 2 - s) sets it
// iff level >= s + 2; neither sum leaves its field.
template <int B>
__device__ __forceinline__ bool fixed_word_invalid(uint32_t w, uint32_t s)
{
    static_assert(B == 4 || B == 8, "fields must tile the word");
    constexpr uint32_t kOnes = B == 4 ? 0x11111111u : 0x01010101u;
    constexpr uint32_t kTop = kOnes << (B - 1), kLevels = kTop - kOnes;
    const uint32_t lv = w & kLevels;
    const uint32_t nonzero = (lv + kLevels) & kTop;
    const uint32_t above = (lv + ((1u << (B - 1)) - 2u - s) * kOnes) & kTop;
    return (above | (w & kTop & ~nonzero)) != 0u;
}

template <int B, bool kLut>
__global__ __launch_bounds__(256) void k_unpack_accumulate_fixed32(UnpackParams P)
{
    __shared__ float tile[256 * 33];                          // a thread's 32 results in a row of 33: no bank conflicts
    extern __shared__ __align__(128) double lut[];            // kLut: [lut_tabs][K][entries]
    constexpr uint32_t kEntries = fixed_lut_entries(B);
    constexpr uint32_t kLevelMask = (1u << (B - 1)) - 1u;
    const uint64_t chunk = (uint64_t)blockIdx.x * 256u + threadIdx.x;
    const uint64_t i0 = chunk * 32u;
    const uint64_t wg0 = (uint64_t)blockIdx.x * 8192u;
    const uint64_t bk_first = P.d <= 0xffffffffull ? (uint64_t)((uint32_t)wg0 / P.bucket) : wg0 / P.bucket;
    if constexpr (kLut) {
        const uint64_t nb = (P.d + P.bucket - 1) / P.bucket;
        const uint32_t total = P.lut_tabs * P.K * kEntries;
        for (uint32_t e = threadIdx.x; e < total; e += 256u) {
            const uint32_t idx = e % kEntries, k = (e / kEntries) % P.K, tab = e / (kEntries * P.K);
            const uint32_t level = B <= 5 ? idx & kLevelMask : idx & 15u, neg = B <= 5 ? idx >> (B - 1) : idx >> 4;
            double val = 0.0;
            if (bk_first + tab < nb && level >= 1u && level <= P.s + 1u) {
                val = fixed_level_value(P, (double)P.norms[k][bk_first + tab], level);
                val = neg ? -val : val;
            }
            lut[e] = val;
        }
        __syncthreads();
    }
    double sum[32];
#pragma unroll
    for (int c = 0; c < 32; ++c)
        sum[c] = 0.0;
    bool bad = false;
    if (i0 < P.d) {
        const uint64_t bk = P.d <= 0xffffffffull ? (uint64_t)((uint32_t)i0 / P.bucket) : i0 / P.bucket;
        const uint32_t j0 = (uint32_t)(i0 - bk * P.bucket);
        const uint64_t word0 = bk * P.wpb + (uint64_t)(j0 / 32u) * B;
        const double *tab = lut + (uint32_t)(bk - bk_first) * P.K * kEntries;
        for (uint32_t k = 0; k < P.K; ++k) {
            const uint32_t *f = P.packed[k] + word0;
            uint32_t w[B];
#pragma unroll
            for (int t = 0; t < B; ++t)
                w[t] = f[t];
            double nrm = 0.0;
            if constexpr (!kLut)
                nrm = (double)P.norms[k][bk];
#pragma unroll
            for (int c = 0; c < 32; ++c) {
                // code c occupies bits [c*B, c*B + B) of the B words, most significant bit first
                const int bit = c * B, wi = bit >> 5, off = bit & 31;
                uint32_t code;
                if (off + B <= 32)
                    code = (w[wi] >> (32 - off - B)) & ((1u << B) - 1u);
                else
                    code = ((w[wi] << (off + B - 32)) | (w[wi + 1 < B ? wi + 1 : wi] >> (64 - off - B))) & ((1u << B) - 1u);
                if constexpr (kLut) {
                    const uint32_t level = code & kLevelMask;
                    bad |= level > P.s + 1u || code == (1u << (B - 1));
                    sum[c] += tab[k * kEntries + fixed_lut_index<B>(code)];
                } else {
                    const uint32_t level = code & kLevelMask, neg = code >> (B - 1);
                    bad |= level > P.s + 1u || (level == 0u && neg);
                    if (level) {
                        const double val = fixed_level_value(P, nrm, min(level, 15u));
                        sum[c] += neg ? -val : val;
                    }
                }
            }
        }
    }
    if (bad)
        atomicOr(P.flags, kFlagMalformed);
    const double sc = (double)P.scale;
#pragma unroll
    for (int c = 0; c < 32; ++c)
        tile[threadIdx.x * 33u + (uint32_t)c] = (float)(sc * sum[c]);
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * 8192u;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const uint32_t e = ((uint32_t)it * 256u + threadIdx.x) * 4u;          // element of the workgroup's 8192
        const uint64_t i = base + e;
        if (i >= P.d)
            continue;
        const float *row = tile + (e >> 5) * 33u + (e & 31u);
        float4 o{row[0], row[1], row[2], row[3]};
        if (i + 3u < P.d) {
            if (P.accumulate) {
                const float4 prev = *reinterpret_cast<const float4 *>(P.out + i);
                o.x += prev.x;
                o.y += prev.y;
                o.z += prev.z;
                o.w += prev.w;
            }
            *reinterpret_cast<float4 *>(P.out + i) = o;
        } else {
            const float r[4] = {o.x, o.y, o.z, o.w};
            for (uint32_t c = 0; c < 4u && i + c < P.d; ++c)
                P.out[i + c] = P.accumulate ? P.out[i + c] + r[c] : r[c];
        }
    }
}

// ---- 4 and 8 bits: one word per worker and thread, whole lines out -----------------------------------------------
// A thread's sums are of whole float4 groups that lie side by side over the wave, so the results leave in full lines
// without a trip through LDS, and a thread holds 8 (4) fp64 sums instead of 32: eight waves per SIMD instead of three.
// At 8 bits a word is four coordinates = one group.  At 4 bits it is eight, and a wave's 64 words are two rows of 64
// groups: even lanes load the words of the first row, odd lanes those of the second, and a lane pair trades halves, after
// which each lane holds the codes of its group of the first row (top half) and of the second.
// K = 8, 25.6 M coordinates, 4 bits: 52 us with k_unpack_accumulate_fixed32 (bound by the loads in flight of three waves
// per SIMD and by LDS), 39 us with this.
constexpr uint32_t kUnpackIters = 4;
constexpr uint32_t unpack_direct_coords(uint32_t b) { return kUnpackIters * 256u * (b == 4u ? 8u : 4u); }   // per workgroup

// kOneBucket: what a wave handles at a time (512 or 256 coordinates) never crosses a bucket boundary.  kFew: one or two
// workers, whose words of all iterations are requested at once: a wave with one or two words in flight is too little for
// the memory.  8 bits, 40 M coordinates of one worker: 37.5 us in turn, 28.1 at once (k_unpack_accumulate_fixed32 31.4); of
// two 43.1, 36.2 (40.3); three fill it (48.7 against 60.9).  4 bits move half as much and gain nothing (28.9 to 30.5 in
// turn, 30.0 at once).
template <int B, bool kOneBucket, bool kFew = false>
__global__ __launch_bounds__(256) void k_unpack_accumulate_fixed_direct(UnpackParams P)
{
    static_assert(B == 4 || B == 8, "a word is whole groups of four codes");
    extern __shared__ __align__(128) double lut[];            // [lut_tabs][K][entries], as in k_unpack_accumulate_fixed32
    constexpr uint32_t kEntries = fixed_lut_entries(B);
    constexpr uint32_t kGroups = B == 4 ? 2u : 1u;            // float4 groups per lane and iteration
    constexpr uint32_t kWaveCoords = 256u * kGroups;
    const uint32_t lane = threadIdx.x & (kWave - 1u), wave = uniform_u32(threadIdx.x / kWave);
    const uint64_t wg0 = (uint64_t)blockIdx.x * unpack_direct_coords(B);
    auto bucket_of = [&](uint64_t i) { return P.d <= 0xffffffffull ? (uint64_t)((uint32_t)i / P.bucket) : i / P.bucket; };
    const uint64_t bk_first = bucket_of(wg0);
    {
        const uint64_t nb = (P.d + P.bucket - 1) / P.bucket;
        const uint32_t total = P.lut_tabs * P.K * kEntries;
        for (uint32_t e = threadIdx.x; e < total; e += 256u) {
            const uint32_t idx = e % kEntries, k = (e / kEntries) % P.K, tab = e / (kEntries * P.K);
            const uint32_t level = B == 4 ? idx & 7u : idx & 15u, neg = B == 4 ? idx >> 3 : idx >> 4;
            double val = 0.0;
            if (bk_first + tab < nb && level >= 1u && level <= P.s + 1u) {
                val = fixed_level_value(P, (double)P.norms[k][bk_first + tab], level);
                val = neg ? -val : val;
            }
            lut[e] = val;
        }
        __syncthreads();
    }
    const uint32_t wsel = B == 4 ? (lane & 1u) * 32u + (lane >> 1) : lane;       // which of the wave's words this lane loads
    const uint32_t swap = lane & 1u ? 0x05040100u : 0x03020706u;                 // halves of (other lane's, own)
    const double sc = (double)P.scale;
    bool bad = false;
    auto first_of_wave = [&](uint32_t it) { return wg0 + (uint64_t)(it * 4u + wave) * kWaveCoords; };
    auto first_of_word = [&](uint64_t c_wave) { return c_wave + wsel * (32u / B); };    // (of this lane's word)
    // returns the word's index; tab: LDS index of the table of (bucket of group, worker 0)
    auto place = [&](uint64_t c_wave, uint32_t (&tab)[kGroups]) {
        const uint64_t c_word = first_of_word(c_wave);
        const uint64_t bk = bucket_of(kOneBucket ? c_wave : c_word);
#pragma unroll
        for (uint32_t g = 0; g < kGroups; ++g)                // (a group beyond the end: any table inside)
            tab[g] = (uint32_t)((kOneBucket ? bk : bucket_of(min(c_wave + 256u * g + 4u * lane, P.d - 1u))) - bk_first) * P.K *
                     kEntries;
        return bk * P.wpb + (uint32_t)(c_word - bk * P.bucket) / (32u / B);
    };
    uint32_t ahead[kFew ? kUnpackIters : 1][2], tabs[kFew ? kUnpackIters : 1][kGroups];
    if constexpr (kFew) {
#pragma unroll
        for (uint32_t it = 0; it < kUnpackIters; ++it) {
            const uint64_t c_wave = first_of_wave(it);
            ahead[it][0] = ahead[it][1] = 0u;
            if (c_wave < P.d) {
                const uint64_t word = place(c_wave, tabs[it]);
                if (first_of_word(c_wave) < P.d) {
                    ahead[it][0] = P.packed[0][word];
                    if (P.K > 1u)
                        ahead[it][1] = P.packed[1][word];
                }
            }
        }
    }
#pragma unroll(kFew ? kUnpackIters : 1)
    for (uint32_t it = 0; it < kUnpackIters; ++it) {
        const uint64_t c_wave = first_of_wave(it);
        if (c_wave >= P.d)
            break;
        uint64_t word = 0;
        uint32_t tab[kGroups];
        if constexpr (kFew) {
#pragma unroll
            for (uint32_t g = 0; g < kGroups; ++g)
                tab[g] = tabs[it][g];
        } else {
            word = place(c_wave, tab);
        }
        const bool live = first_of_word(c_wave) < P.d;
        double sum[4 * kGroups];
#pragma unroll
        for (uint32_t c = 0; c < 4u * kGroups; ++c)
            sum[c] = 0.0;
        constexpr uint32_t kFlight = kFew ? 2u : 8u;
        for (uint32_t k0 = 0; k0 < (kFew ? 1u : P.K); k0 += kFlight) {
            uint32_t w[kFlight];
#pragma unroll
            for (uint32_t q = 0; q < kFlight; ++q) {
                if constexpr (kFew) {
                    w[q] = ahead[it][q];
                } else {
                    w[q] = 0u;
                    if (k0 + q < P.K && live)
                        w[q] = P.packed[k0 + q][word];
                }
            }
#pragma unroll
            for (uint32_t q = 0; q < kFlight; ++q) {
                if (k0 + q >= P.K)                            // uniform
                    break;
                bad |= fixed_word_invalid<B>(w[q], P.s);
                uint32_t x = w[q];
                if constexpr (B == 4)
                    x = __builtin_amdgcn_perm((uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xf, 0xf, true), x, swap);
#pragma unroll
                for (uint32_t c = 0; c < 4u * kGroups; ++c) {
                    const uint32_t code = (x >> (32u - B - c * B)) & ((1u << B) - 1u);
                    sum[c] += lut[tab[c / 4u] + (k0 + q) * kEntries + fixed_lut_index<B>(code)];
                }
            }
        }
#pragma unroll
        for (uint32_t g = 0; g < kGroups; ++g) {
            const uint64_t i = c_wave + 256u * g + 4u * lane;
            float4 o{(float)(sc * sum[4 * g]), (float)(sc * sum[4 * g + 1]), (float)(sc * sum[4 * g + 2]),
                     (float)(sc * sum[4 * g + 3])};
            if (i + 3u < P.d) {
                float4 *const dst = reinterpret_cast<float4 *>(P.out + i);
                if (P.accumulate) {
                    const float4 prev = *dst;
                    *dst = float4{o.x + prev.x, o.y + prev.y, o.z + prev.z, o.w + prev.w};
                } else {
                    store_once4(dst, o);
                }
            } else {
                const float r[4] = {o.x, o.y, o.z, o.w};
                for (uint32_t c = 0; c < 4u && i + c < P.d; ++c)
                    P.out[i + c] = P.accumulate ? P.out[i + c] + r[c] : r[c];
            }
        }
    }
    if (bad)
        atomicOr(P.flags, kFlagMalformed);
}

// Any bucket size: one coordinate per thread.
__global__ __launch_bounds__(256) void k_unpack_accumulate_fixed1(UnpackParams P)
{
    const uint64_t i0 = (uint64_t)blockIdx.x * 256u + threadIdx.x;
    if (i0 >= P.d)
        return;
    const uint64_t bk = i0 / P.bucket;
    const uint32_t j0 = (uint32_t)(i0 - bk * P.bucket);
    const uint32_t bit0 = j0 * P.b;
    const uint32_t wi = bit0 >> 5, sh = bit0 & 31u;
    const bool two = sh + P.b > 32u;                        // the code straddles a word boundary
    const uint32_t mask_level = (1u << (P.b - 1u)) - 1u;
    double sum = 0.0;
    bool bad = false;
    for (uint32_t k = 0; k < P.K; ++k) {
        const uint32_t *f = P.packed[k] + bk * P.wpb + wi;
        const uint32_t w0 = f[0];
        const uint32_t w1 = two ? f[1] : 0u;
        const uint64_t win = (((uint64_t)w0 << 32) | w1) << sh;     // the code on top
        const uint32_t code = (uint32_t)(win >> (64u - P.b));
        const uint32_t level = code & mask_level, neg = code >> (P.b - 1u);
        bad |= level > P.s + 1u || (level == 0u && neg);
        if (level) {
            const double val = fixed_level_value(P, (double)P.norms[k][bk], min(level, 15u));
            sum += neg ? -val : val;
        }
    }
    if (bad)
        atomicOr(P.flags, kFlagMalformed);
    const float r = (float)((double)P.scale * sum);
    P.out[i0] = P.accumulate ? P.out[i0] + r : r;
}

}  // namespace nuq
