// Huffman-coded levels (Sec. 5, "Efficient Encoding": a Huffman code for the level indices, built from a sample and
// then kept).  Message of the level|sign bytes: per bucket, for every coordinate in order, the canonical codeword of
// its level index (most significant bit first), then its sign bit when the level is not zero; bit_off, words and
// word alignment as for the ERC strings; sync entry (b, g) = bit offset, from the bucket's start, of coordinate
// g * stride (the bucket's bit length if the bucket ends before it).
#pragma once

#include "nuq_decode_kernels.hpp"
#include "nuq_encode_kernels.hpp"

namespace nuq {

// A canonical code over the level indices 0..s+1 (at most 16 symbols, lengths 1..15).
struct HuffmanCode {
    uint32_t code[16];     // codeword of a symbol, right-aligned
    uint32_t len[16];      // its length
    uint32_t first[16];    // by length L: first codeword of that length
    uint32_t count[16];    // number of codewords of that length
    uint32_t offset[16];   // index into `sorted` of the first symbol of that length
    uint32_t sorted[16];   // symbols by (length, symbol)
    uint32_t maxlen;
    uint32_t nsym;
};

// ---------------------------------------------------------------------------- histogram
__global__ __launch_bounds__(256) void k_level_histogram(const uint8_t *q, uint64_t d, unsigned long long *hist)
{
    __shared__ uint32_t local[128];
    if (threadIdx.x < 128u)
        local[threadIdx.x] = 0u;
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (uint64_t i = (uint64_t)blockIdx.x * 256u + threadIdx.x; i < d; i += stride)
        atomicAdd(&local[q[i] & 0x7fu], 1u);
    __syncthreads();
    if (threadIdx.x < 16u && local[threadIdx.x])
        atomicAdd(&hist[threadIdx.x], (unsigned long long)local[threadIdx.x]);
    // level indices above 15 cannot be coded; they are counted nowhere and rejected by the encoder
}

__global__ void k_zero_u64(unsigned long long *p, uint32_t n)
{
    if (threadIdx.x < n)
        p[threadIdx.x] = 0ull;
}

// ------------------------------------------------------------------- bucket bit lengths
// lens[b] = sum over the bucket of len[level] + (level != 0).  One bucket per team, bytes read as in the encoders.
template <int TEAM, int VPT>
__global__ __launch_bounds__(TeamGeom<TEAM>::kWG) void k_huffman_lens(EncodeParams P, EncodeBatch Wk, HuffmanCode H)
{
    __shared__ uint32_t scratch_all[TeamGeom<TEAM>::kTeamsPerWG][16];
    const EncodeWorker &W = Wk.w[0];
    const uint32_t tid = threadIdx.x % TEAM;
    const uint32_t team = threadIdx.x / TEAM;
    const uint64_t b = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG + team;
    const bool active = b < P.nb;
    const uint64_t base = active ? b * P.bucket : 0;
    const uint32_t nbk = active ? (uint32_t)min((uint64_t)P.bucket, P.d - base) : 0u;
    const uint8_t *qg = W.q_in + base;
    uint32_t bits = 0;
    bool bad = false;
    for (uint32_t c = tid; c < nbk; c += TEAM) {
        const uint32_t byte = qg[c], level = byte & 0x7fu;
        bad |= level > P.s + 1u || (level == 0u && byte);
        bits += H.len[min(level, 15u)] + (level ? 1u : 0u);
    }
    if (bad)
        atomicOr(P.flags, kFlagMalformed);
    uint32_t total;
    team_exclusive_sum<TEAM>(bits, scratch_all[team], total);
    if (active && tid == 0)
        P.units[b] = total;                 // (bits here: k_chunk_sums and k_bit_offsets of this path take bits)
}

// bit_off from lens: one workgroup per chunk of 1024 buckets, chunk_prefix[c] = words before the chunk.
__global__ __launch_bounds__(256) void k_bit_offsets(const uint32_t *lens, uint64_t nb, const uint64_t *chunk_prefix,
                                                     uint64_t *bit_off)
{
    __shared__ uint32_t wave_tot[4];
    const uint64_t b0 = (uint64_t)blockIdx.x * kChunk + threadIdx.x * 4u;
    uint32_t len[4], wc[4], mine = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        len[i] = b0 + i < nb ? lens[b0 + i] : 0u;
        wc[i] = (len[i] + 31u) >> 5;
        mine += wc[i];
    }
    uint32_t inc = mine;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = (uint32_t)__shfl_up((int)inc, off, 64);
        if (lane >= off)
            inc += t;
    }
    if (lane == 63)
        wave_tot[wave] = inc;
    __syncthreads();
    uint64_t start = chunk_prefix[blockIdx.x] + inc - mine;
    for (int w = 0; w < wave; ++w)
        start += wave_tot[w];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (b0 + i < nb)
            bit_off[b0 + i + 1] = 32ull * start + len[i];
        start += wc[i];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0)
        bit_off[0] = 0;
}

// --------------------------------------------------------------------------------- emit
// LDS words per team: [qb32: rows * TEAM][field: worst case ceil(bucket * 16 / 32) + 1][sync: nsync][scratch: 64]
__host__ __device__ inline uint32_t huffman_lds_words(uint32_t rows, uint32_t team, uint32_t bucket, uint32_t nsync)
{
    const uint32_t w = (rows * team + (bucket + 1u) / 2u + 1u + nsync + 1u) & ~1u;
    return w + 64u;
}

// What a level|sign byte sends: bits = codeword of min(byte & 0x7f, 15), then the sign bit when the level is not zero;
// entry = length << 24 | bits.  256 entries, built once per workgroup (the codeword tables are kernel arguments: a
// lookup by a per-lane index there is a memory access; this table is an LDS read).
template <uint32_t WG>
__device__ __forceinline__ void huffman_byte_table(const HuffmanCode &H, uint32_t *enc)
{
    for (uint32_t p = threadIdx.x; p < 256u; p += WG) {
        const uint32_t level = min(p & 0x7fu, 15u);
        uint32_t n = H.len[level], v = H.code[level];
        if (level) {
            v = (v << 1) | (p >> 7);
            ++n;
        }
        enc[p] = (n << 24) | v;
    }
}

// The bucket's bit string from its level|sign bytes in LDS (qb32) into the zeroed LDS words `field`, sync offsets
// into sync_l; returns the bucket's bit length to every thread.  Each thread codes a contiguous chunk of rows * 4
// coordinates: codewords (looked up by byte in `enc`) are shifted into a 64-bit register and leave it 32 bits at a
// time, OR-ed into the field (a chunk's first and last words are shared with its neighbours).
template <int TEAM>
__device__ __forceinline__ uint32_t huffman_from_lds(const EncodeParams &P, const uint32_t *enc, const uint32_t *qb32,
                                                     uint32_t *field, uint32_t *sync_l, uint32_t *scratch,
                                                     uint32_t nbk, uint32_t tid)
{
    const uint32_t per = P.rows * 4u;
    const uint32_t c0 = min(tid * per, nbk), c1 = min(c0 + per, nbk);
    const uint32_t *qw = qb32 + (c0 >> 2);              // c0 is a multiple of four, or nbk (then the chunk is empty)
    const uint32_t nfull = (c1 - c0) >> 2, ntail = (c1 - c0) & 3u;
    uint32_t bits = 0;
    // Four level-0 coordinates in a word (three words in four on sparse gradients) are coded in one go when their
    // codewords fit the register's spare 16 bits.
    const uint32_t e0 = enc[0], len0 = e0 >> 24, code0 = e0 & 0xffffffu;
    const bool quad = len0 <= 4u;
    const uint32_t code0x4 = quad ? ((code0 << (3u * len0)) | (code0 << (2u * len0)) | (code0 << len0) | code0) : 0u;
    for (uint32_t i = 0; i < nfull; ++i) {
        const uint32_t w = qw[i];
        if (w == 0u)
            bits += 4u * len0;
        else
            bits += (enc[w & 0xffu] >> 24) + (enc[(w >> 8) & 0xffu] >> 24) + (enc[(w >> 16) & 0xffu] >> 24) +
                    (enc[w >> 24] >> 24);
    }
    if (ntail) {
        const uint32_t w = qw[nfull];
        for (uint32_t j = 0; j < ntail; ++j)
            bits += enc[(w >> (8u * j)) & 0xffu] >> 24;
    }
    uint32_t total;
    uint32_t pos = team_exclusive_sum<TEAM>(bits, scratch, total);
    const uint32_t nwords = (total + 31u) >> 5;
    for (uint32_t i = tid; i < nwords; i += TEAM)
        field[i] = 0u;
    for (uint32_t i = tid; i < P.nsync; i += TEAM)
        sync_l[i] = total;                          // boundaries at or beyond the bucket's end
    team_barrier<TEAM>();

    if (c0 < c1) {
        uint32_t wi = pos >> 5, fill = pos & 31u;
        uint64_t acc = 0;
        const uint32_t smask = P.sync_shift ? (1u << P.sync_shift) - 1u : 0u;
        auto push = [&](uint32_t v, uint32_t n) {       // n <= 16: at most 31 + 16 bits are pending
            acc = (acc << n) | v;
            fill += n;
            pos += n;
            if (fill >= 32u) {
                fill -= 32u;
                atomicOr(&field[wi++], (uint32_t)(acc >> fill));
                acc &= (1ull << fill) - 1ull;
            }
        };
        auto put = [&](uint32_t byte) {
            const uint32_t e = enc[byte];
            push(e & 0xffffffu, e >> 24);
        };
        for (uint32_t i = 0; i <= nfull; ++i) {
            if (i == nfull && !ntail)
                break;
            // a sync boundary is a multiple of 32 coordinates, so only a word's first coordinate can be one
            const uint32_t w = qw[i], c = c0 + 4u * i;
            if (P.sync_shift && c && (c & smask) == 0u)
                sync_l[(c >> P.sync_shift) - 1u] = pos;
            if (i == nfull) {
                for (uint32_t j = 0; j < ntail; ++j)
                    put((w >> (8u * j)) & 0xffu);
            } else if (w == 0u && quad) {
                push(code0x4, 4u * len0);
            } else {
                put(w & 0xffu);
                put((w >> 8) & 0xffu);
                put((w >> 16) & 0xffu);
                put(w >> 24);
            }
        }
        if (fill)
            atomicOr(&field[wi], (uint32_t)(acc << (32u - fill)));
    }
    return total;
}

// ---- levels up to 7 (s <= 6): two coordinates per table entry ------------------------------------------------------
// A coordinate is then four bits, level | sign << 3, and two of them index a table of 256 entries: what both send (at most
// 16 bits: codewords have at most s + 1 bits) | its length << 16.  A word of four coordinates is two reads and one push of
// up to 32 bits, the same instructions whatever the levels are; byte by byte (huffman_from_lds) a wave went through the way
// for words of zeros and through that for others for nearly every word, 14 instructions per coordinate.  Encode + decode:
// 8 x 25.6 M coordinates at s = 3 252 -> 219 us, 4 x 16.8 M at s = 5 187 -> 154.  From s = 7 on a level has more than three
// bits and huffman_from_lds stays.

// Bytes level | sign << 3 (the sign of a zero means nothing).
struct NibbleBytes {
    __device__ __forceinline__ uint32_t any(uint32_t sg, uint32_t levels) const
    {
        return ((sg >> 4) & 0x08080808u) | levels;
    }
    __device__ __forceinline__ uint32_t first(uint32_t sg, uint32_t tb) const { return any(sg, (tb >> 7) & 0x01010101u); }
    __device__ __forceinline__ uint32_t two(uint32_t sg, uint32_t tb, uint32_t tb2) const
    {
        return first(sg, tb) + ((tb2 >> 7) & 0x01010101u);
    }
};

// The table's entries for this thread (one of 256, or two), in two halves as TableCopy: its codewords requested before the gradient's
// loads, the entry made and stored when those are under way.
template <uint32_t WG>
struct PairTable {
    static constexpr uint32_t kPer = WG < 256u ? 256u / WG : 1u, kStep = 256u / kPer;
    uint32_t len0, code0, len1[kPer], code1[kPer];        // the first coordinate's bits are the same for all of a thread's
    __device__ __forceinline__ explicit PairTable(const HuffmanCode &H)
    {
        len0 = H.len[threadIdx.x & 7u];
        code0 = H.code[threadIdx.x & 7u];
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i) {
            const uint32_t level = ((threadIdx.x + i * kStep) >> 4) & 7u;
            len1[i] = H.len[level];
            code1[i] = H.code[level];
        }
    }
    __device__ __forceinline__ void store(uint32_t *pairs) const
    {
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i) {
            const uint32_t p = threadIdx.x + i * kStep;
            if (p < 256u) {
                const uint32_t s0 = (p & 7u) ? 1u : 0u, s1 = (p & 0x70u) ? 1u : 0u;    // a sign bit follows
                const uint32_t c0 = (code0 << s0) | (s0 & (p >> 3)), c1 = (code1[i] << s1) | (s1 & (p >> 7));
                pairs[p] = (c0 << (len1[i] + s1)) | c1 | ((len0 + s0 + len1[i] + s1) << 16);
            }
        }
    }
};

// huffman_from_lds for such bytes and that table.  A thread's words are looked up once and kept (VPT of them).
template <int TEAM, int VPT>
__device__ __forceinline__ uint32_t huffman_pairs_from_lds(const EncodeParams &P, const uint32_t *pairs, const uint32_t *qb32,
                                                           uint32_t *field, uint32_t *sync_l, uint32_t *scratch, uint32_t nbk,
                                                           uint32_t tid)
{
    const uint32_t c0 = tid * P.rows * 4u;
    const uint32_t *qw = qb32 + tid * P.rows;
    // the index boundary (a multiple of the stride, 64 or more, so of four) inside this chunk of at most 64 coordinates
    const uint32_t smask = (1u << P.sync_shift) - 1u;
    const uint32_t cb = P.sync_shift ? (c0 + smask) & ~smask : ~0u;
    const bool has_boundary = P.sync_shift && cb && cb < min(c0 + P.rows * 4u, nbk);
    const uint32_t iw = (cb - c0) >> 2;
    uint32_t code[VPT], len[VPT], bits = 0, before = 0;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        code[i] = len[i] = 0;
        if ((uint32_t)i < P.rows) {
            before = (uint32_t)i == iw ? bits : before;
            const uint32_t c = c0 + 4u * (uint32_t)i, w = qw[i];
            if (__all(c + 4u <= nbk)) {
                const uint32_t t = w | (w >> 4);
                const uint32_t e0 = pairs[t & 0xffu], e1 = pairs[(t >> 16) & 0xffu], l1 = e1 >> 16;
                code[i] = ((e0 & 0xffffu) << l1) | (e1 & 0xffffu);
                len[i] = (e0 >> 16) + l1;
            } else {                                              // the bucket ends in some lane's word: one by one
                const uint32_t zero = pairs[0] >> 17;             // length of level 0's codeword
                for (uint32_t j = 0; j < 4u; ++j)
                    if (c + j < nbk) {
                        const uint32_t e = pairs[(w >> (8u * j)) & 15u], l = (e >> 16) - zero;
                        code[i] = (code[i] << l) | ((e & 0xffffu) >> zero);
                        len[i] += l;
                    }
            }
            bits += len[i];
        }
    }
    uint32_t total;
    const uint32_t pos = team_exclusive_sum<TEAM>(bits, scratch, total);
    const uint32_t nwords = (total + 31u) >> 5;
    for (uint32_t i = 4u * tid; i < nwords; i += 4u * TEAM)
        *reinterpret_cast<uint4 *>(field + i) = uint4{0u, 0u, 0u, 0u};
    for (uint32_t i = tid; i < P.nsync; i += TEAM)
        sync_l[i] = total;                          // boundaries at or beyond the bucket's end
    team_barrier<TEAM>();
    BitWriter out(pos);                             // (at most 31 + 32 bits are pending)
#pragma unroll
    for (int i = 0; i < VPT; ++i)
        if ((uint32_t)i < P.rows)
            out.put(field, code[i], len[i]);
    out.flush(field);
    if (has_boundary)
        sync_l[(cb >> P.sync_shift) - 1u] = pos + before;
    return total;
}

// Norms + quantizer + Huffman coding of one bucket per team, v read once, all workers in one launch (blockIdx.y): the
// bit string goes to the staging area and its length where k_finish looks for it (place_bucket); that kernel
// turns them into bit_off and words as for the ERC strings.  kPairs: s <= 6.
template <int TEAM, int VPT, bool kPairs>
__global__ __launch_bounds__(TeamGeom<TEAM>::kWG) void k_huffman_fused(EncodeParams P, EncodeBatch Wk, HuffmanCode H)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const EncodeWorker &W = Wk.w[blockIdx.y];
    const uint32_t tid = threadIdx.x % TEAM;
    const uint32_t team = team_uniform_u32<TEAM>(threadIdx.x / TEAM);
    uint32_t *lds = smem + team * P.lds_words;
    uint32_t *qb32 = lds;
    uint32_t *field = qb32 + P.rows * TEAM;
    uint32_t *sync_l = field + P.out_cap;
    uint32_t *scratch = lds + P.lds_words - 64u;
    const EncodeOut O = encode_out<TEAM>(P, W);
    const uint64_t b = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG + team;
    const bool active = b < P.nb;
    const uint64_t base = active ? b * P.bucket : 0;
    const uint32_t nbk = active ? (uint32_t)min((uint64_t)P.bucket, P.d - base) : 0u;
    __shared__ uint32_t enc[256];
    uint32_t total;
    if constexpr (kPairs) {
        const PairTable<TeamGeom<TEAM>::kWG> table(H);
        front_quantize_to_lds<TEAM, VPT>(P, W, b, active, base, nbk, tid, qb32, scratch, NibbleBytes{},
                                         [&] { table.store(enc); });
        __syncthreads();
        total = huffman_pairs_from_lds<TEAM, VPT>(P, enc, qb32, field, sync_l, scratch, nbk, tid);
    } else {
        huffman_byte_table<TeamGeom<TEAM>::kWG>(H, enc);
        front_quantize_to_lds<TEAM, VPT>(P, W, b, active, base, nbk, tid, qb32, scratch, PlainBytes{}, [] {});
        __syncthreads();
        total = huffman_from_lds<TEAM>(P, enc, qb32, field, sync_l, scratch, nbk, tid);
    }
    uint32_t *slot = O.unit;
    if constexpr (TeamGeom<TEAM>::kTeamsPerWG > 1) {
        __shared__ UnitWords<TEAM> unit_words;
        announce_bucket<TEAM>(unit_words, active, total);
        __syncthreads();
        slot = place_bucket<TEAM>(unit_words, O, active, b, total);
    } else {
        team_barrier<TEAM>();
    }
    if (active) {
        store_bucket<TEAM>(slot, field, (total + 31u) >> 5, tid);
        uint32_t *sg = O.sync + b * P.nsync;
        for (uint32_t i = tid; i < P.nsync; i += TEAM)
            sg[i] = sync_l[i];
    }
    if constexpr (TeamGeom<TEAM>::kTeamsPerWG == 1)
        report_length(O, b, total, tid);
}

template <int TEAM, int VPT>
__global__ __launch_bounds__(TeamGeom<TEAM>::kWG) void k_huffman_emit(EncodeParams P, EncodeBatch Wk, HuffmanCode H)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const EncodeWorker &W = Wk.w[0];
    const uint32_t tid = threadIdx.x % TEAM;
    const uint32_t team = team_uniform_u32<TEAM>(threadIdx.x / TEAM);
    uint32_t *lds = smem + team * P.lds_words;
    uint32_t *qb32 = lds;
    uint32_t *field = qb32 + P.rows * TEAM;
    uint32_t *sync_l = field + (P.bucket + 1u) / 2u + 1u;
    uint32_t *scratch = lds + P.lds_words - 64u;
    const uint64_t b = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG + team;
    const bool active = b < P.nb;
    const uint64_t base = active ? b * P.bucket : 0;
    const uint32_t nbk = active ? (uint32_t)min((uint64_t)P.bucket, P.d - base) : 0u;
    __shared__ uint32_t enc[256];
    huffman_byte_table<TeamGeom<TEAM>::kWG>(H, enc);
    front_bytes_to_lds<TEAM, VPT>(P, W, base, nbk, tid, qb32);
    __syncthreads();

    const uint32_t total = huffman_from_lds<TEAM>(P, enc, qb32, field, sync_l, scratch, nbk, tid);
    const uint32_t nwords = (total + 31u) >> 5;
    team_barrier<TEAM>();
    if (active) {
        const uint64_t start_word = (W.bit_off[b] + 31ull) >> 5;
        const bool fits = start_word + nwords <= W.words_cap;
        if (fits)
            for (uint32_t i = tid; i < nwords; i += TEAM)
                W.words[start_word + i] = field[i];
        else if (tid == 0 && nwords)
            atomicOr(P.flags, kFlagCapacity);
        uint32_t *sg = W.sync + b * P.nsync;
        for (uint32_t i = tid; i < P.nsync; i += TEAM)
            sg[i] = sync_l[i];
    }
}

// ------------------------------------------------------------------------------- decode
struct HuffmanStream {
    const uint64_t *bit_off;
    const uint32_t *words;
    const uint32_t *sync;
    uint8_t *q;
};

struct HuffmanDecodeParams {
    HuffmanStream w[kMaxBatch];      // one per worker: blockIdx.y
    uint32_t *flags;
    uint64_t d;
    uint64_t nb;
    uint32_t bucket;
    uint32_t sync_shift;
    uint32_t nsync;
    uint32_t nseg;
};

// One thread per unit = (bucket, sync segment): walks its codewords and writes level|sign bytes.
__global__ __launch_bounds__(256) void k_huffman_decode(HuffmanDecodeParams P, HuffmanCode H)
{
    const HuffmanStream &W = P.w[blockIdx.y];
    const uint64_t u = (uint64_t)blockIdx.x * 256u + threadIdx.x;
    if (u >= P.nb * P.nseg)
        return;
    const uint64_t b = u / P.nseg;
    const uint32_t g = (uint32_t)(u - b * P.nseg);
    const uint32_t nbk = (uint32_t)min((uint64_t)P.bucket, P.d - b * P.bucket);
    const uint32_t c_lo = P.sync_shift ? g << P.sync_shift : 0u;
    if (c_lo >= nbk)
        return;
    const uint32_t c_hi = P.sync_shift ? min(nbk, (g + 1u) << P.sync_shift) : nbk;
    const uint64_t start = (W.bit_off[b] + 31ull) & ~31ull, end = W.bit_off[b + 1];
    const uint32_t len = end > start ? (uint32_t)(end - start) : 0u;
    const uint32_t *sg = W.sync + b * P.nsync;
    const uint32_t lo = g ? sg[g - 1u] : 0u;
    const uint32_t hi = g + 1u < P.nseg ? sg[g] : len;           // where the next segment starts
    bool bad = lo > hi || hi > len;
    uint8_t *qb = W.q + b * P.bucket;
    if (!bad) {
        WalkWords gw{W.words + (start >> 5)};
        BitReader<WalkWords> br;
        br.init(gw, lo, (len + 31u) >> 5);
        uint32_t pos = lo;
        for (uint32_t c = c_lo; c < c_hi; ++c) {
            br.refill();
            const uint32_t w = br.peek();
            uint32_t L = 1, sym = 0;
            bool found = false;
            for (; L <= H.maxlen; ++L) {
                const uint32_t idx = (w >> (32u - L)) - H.first[L];
                if (idx < H.count[L]) {
                    sym = H.sorted[H.offset[L] + idx];
                    found = true;
                    break;
                }
            }
            const uint32_t n = L + (sym ? 1u : 0u);
            if (!found || pos + n > hi) {
                bad = true;
                break;
            }
            const uint32_t neg = sym ? (w >> (31u - L)) & 1u : 0u;
            qb[c] = (uint8_t)(sym | (neg << 7));
            br.skip(n);
            pos += n;
        }
        bad |= pos != hi;
    }
    if (bad)
        atomicOr(P.flags, kFlagMalformed);
}

// Words of a unit's bit string that a lane stages in LDS (a unit of S coordinates at up to two bits per coordinate
// and a little more; longer ones are read from global memory as they go) and the stride of a lane's staging row.
__host__ __device__ inline uint32_t huffman_stage_cap(uint32_t S) { return S / 16u + 6u; }
__host__ __device__ inline uint32_t huffman_stage_stride(uint32_t S) { return huffman_stage_cap(S) + 3u; }   // odd

// The same for messages with a sync index: a wave owns 64 consecutive units.  Code tables and a lookup table on the
// next eight bits (symbol | length << 4; 0 for longer codewords, which take the length-by-length walk) live in LDS.
// A lane first copies its unit's words into its staging row (independent loads, all in flight together), then
// parses them with the window of the ERC decoder: position + 31 is the loop variable, the 32-bit window comes from
// two words through one funnel shift, and those two words and the one after them wait in registers (a codeword and
// its sign are at most 16 bits: the pair moves on by one word at most).  Bytes are assembled four at a time into the
// lane's row of an LDS tile (row stride S + 4 bytes: the lanes hit different banks), and the tile goes out unit by
// unit with whole-wave stores.
__global__ __launch_bounds__(64) void k_huffman_decode_tile(HuffmanDecodeParams P, HuffmanCode H)
{
    extern __shared__ __align__(16) uint32_t tile[];            // 64 rows of S / 4 + 1 words, then 64 staging rows
    __shared__ uint8_t lut8[256];
    __shared__ uint32_t first[16], count[16], offset[16], sorted[16];
    __shared__ uint32_t unit_dst_lo[64], unit_dst_hi[64], unit_len[64];
    const uint32_t lane = threadIdx.x;
    const uint32_t S = 1u << P.sync_shift;
    const uint32_t row_words = S / 4u + 1u;
    if (lane < 16u) {
        first[lane] = H.first[lane];
        count[lane] = H.count[lane];
        offset[lane] = H.offset[lane];
        sorted[lane] = H.sorted[lane];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t p = lane; p < 256u; p += 64u) {               // the codeword that starts the eight bits p, if any
        uint32_t entry = 0;
        for (uint32_t L = 1; L <= 8u && L <= H.maxlen; ++L) {
            const uint32_t idx = (p >> (8u - L)) - first[L];
            if (idx < count[L]) {
                entry = sorted[offset[L] + idx] | (L << 4);
                break;
            }
        }
        lut8[p] = (uint8_t)entry;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();

    const HuffmanStream &W = P.w[blockIdx.y];
    const uint64_t u = (uint64_t)blockIdx.x * 64u + lane;
    const bool live = u < P.nb * P.nseg;
    const uint64_t b = live ? u / P.nseg : 0;
    const uint32_t g = live ? (uint32_t)(u - b * P.nseg) : 0u;
    const uint32_t nbk = (uint32_t)min((uint64_t)P.bucket, P.d - b * P.bucket);
    const uint32_t c_lo = g << P.sync_shift;
    const uint32_t c_hi = live && c_lo < nbk ? min(nbk, c_lo + S) : c_lo;      // an empty range for idle lanes
    uint32_t *row = tile + lane * row_words;
    const uint32_t cap = huffman_stage_cap(S), stride = huffman_stage_stride(S);
    uint32_t *srow = tile + 64u * row_words + lane * stride;    // srow[1 + j] = word j of the unit's frame
    bool bad = false;
    if (c_lo < c_hi) {
        const uint64_t start = (W.bit_off[b] + 31ull) & ~31ull, end = W.bit_off[b + 1];
        const uint32_t len = end > start ? (uint32_t)(end - start) : 0u;
        const uint32_t *sg = W.sync + b * P.nsync;
        const uint32_t lo = g ? sg[g - 1u] : 0u;
        const uint32_t hi = g + 1u < P.nseg ? sg[g] : len;
        bad = lo > hi || hi > len;
        const uint32_t w0 = lo >> 5, nw = bad ? 0u : ((hi + 31u) >> 5) - w0;
        if (!bad && nw <= cap) {
            const uint32_t *src = W.words + (start >> 5) + w0;
            for (uint32_t j0 = 0; j0 < nw; j0 += 8u) {
                uint32_t t[8];
#pragma unroll
                for (uint32_t j = 0; j < 8u; ++j)
                    t[j] = src[min(j0 + j, nw - 1u)];
#pragma unroll
                for (uint32_t j = 0; j < 8u; ++j)
                    if (j0 + j < nw)
                        srow[1u + j0 + j] = t[j];
            }
            const uint32_t bit0 = lo & 31u;
            uint32_t p31 = bit0 + 31u, q = p31 >> 5;
            uint32_t hw = srow[q], lw = srow[q + 1u], nx = srow[q + 2u];
            uint32_t four = 0;
            for (uint32_t c = c_lo; c < c_hi; ++c) {
                const uint32_t w = __builtin_amdgcn_alignbit(hw, lw, ~p31);
                uint32_t entry = lut8[w >> 24];
                if (!entry) {                                   // a codeword of nine bits or more (rare), or none
                    for (uint32_t L = 9; L <= H.maxlen; ++L) {
                        const uint32_t idx = (w >> (32u - L)) - first[L];
                        if (idx < count[L]) {
                            entry = sorted[offset[L] + idx] | (L << 4);
                            break;
                        }
                    }
                }
                const uint32_t sym = entry & 15u, L = entry >> 4;
                bad |= !L;
                const uint32_t neg = sym ? (w >> (31u - L)) & 1u : 0u;
                four |= (sym | (neg << 7)) << (8u * (c & 3u));
                if ((c & 3u) == 3u) {
                    row[(c - c_lo) >> 2] = four;
                    four = 0;
                }
                p31 += L + (sym ? 1u : 0u);
                const uint32_t qn = p31 >> 5;
                const bool moved = qn != q;
                hw = moved ? lw : hw;
                lw = moved ? nx : lw;
                q = qn;
                nx = srow[min(qn + 2u, stride - 1u)];
            }
            if ((c_hi - c_lo) & 3u)
                row[(c_hi - c_lo) >> 2] = four;
            bad |= lo - bit0 + (p31 - 31u) != hi;
        } else if (!bad) {
            WalkWords gw{W.words + (start >> 5)};
            BitReader<WalkWords> br;
            br.init(gw, lo, (len + 31u) >> 5);
            uint32_t pos = lo, four = 0;
            for (uint32_t c = c_lo; c < c_hi; ++c) {
                br.refill();
                const uint32_t w = br.peek();
                uint32_t entry = lut8[w >> 24];
                if (!entry) {                                   // a codeword of nine bits or more (rare), or none
                    for (uint32_t L = 9; L <= H.maxlen; ++L) {
                        const uint32_t idx = (w >> (32u - L)) - first[L];
                        if (idx < count[L]) {
                            entry = sorted[offset[L] + idx] | (L << 4);
                            break;
                        }
                    }
                }
                const uint32_t sym = entry & 15u, L = entry >> 4;
                const uint32_t n = L + (sym ? 1u : 0u);
                if (!L || pos + n > hi) {
                    bad = true;
                    break;
                }
                const uint32_t neg = sym ? (w >> (31u - L)) & 1u : 0u;
                four |= (sym | (neg << 7)) << (8u * (c & 3u));
                if ((c & 3u) == 3u) {
                    row[(c - c_lo) >> 2] = four;
                    four = 0;
                }
                br.skip(n);
                pos += n;
            }
            if ((c_hi - c_lo) & 3u)
                row[(c_hi - c_lo) >> 2] = four;                 // a short last segment that is no multiple of four
            bad |= pos != hi;
        }
    }
    if (bad)
        atomicOr(P.flags, kFlagMalformed);
    const uint64_t dst = b * P.bucket + c_lo;
    unit_dst_lo[lane] = (uint32_t)dst;
    unit_dst_hi[lane] = (uint32_t)(dst >> 32);
    unit_len[lane] = c_hi - c_lo;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t i = 0; i < 64u; ++i) {
        const uint32_t n = unit_len[i];
        if (!n)
            continue;
        uint8_t *out = W.q + (((uint64_t)unit_dst_hi[i] << 32) | unit_dst_lo[i]);
        const uint32_t *src = tile + i * row_words;
        if ((reinterpret_cast<uintptr_t>(out) & 3u) == 0) {
            for (uint32_t w4 = lane; w4 < n / 4u; w4 += 64u)
                reinterpret_cast<uint32_t *>(out)[w4] = src[w4];
            for (uint32_t c = (n & ~3u) + lane; c < n; c += 64u)
                out[c] = (uint8_t)(src[c >> 2] >> (8u * (c & 3u)));
        } else {
            for (uint32_t c = lane; c < n; c += 64u)
                out[c] = (uint8_t)(src[c >> 2] >> (8u * (c & 3u)));
        }
    }
}

// The decoder for the usual geometry (buckets and byte arrays that are multiples of 16: every unit starts on a 16-byte
// boundary): as k_huffman_decode_tile, but a lane collects its bytes in registers and stores them itself, 64
// consecutive bytes at a time (ByteSink).  Without the tile a wave needs 6.4 KB of LDS instead of 23, so several
// times as many waves hide each other's latencies (the parse is one dependent chain per lane).
//
// The parse is bound by instruction issue, so it takes several symbols per step: `multi` maps the next eight bits of
// the string to the symbols that end inside them (codeword plus sign bit; up to eight level-0 symbols), their
// count and the running total of their lengths.  An entry with no symbol (a codeword of eight bits or more, or none)
// falls back to one symbol from the 32-bit window.  The bits after a unit's end are the next unit's (or padding
// that reads as level-0 symbols): near the end only as many of an entry's symbols as the unit still has are taken,
// with the length the running total gives, so every step of every lane goes the same way.
constexpr uint32_t kHuffmanDirectWG = 256;

struct MultiEntry {
    uint32_t bytes_lo, bytes_hi;   // level|sign bytes of the symbols, first symbol in the lowest byte, rest zero
    uint32_t count;                // symbols, 0..8
    uint32_t cum;                  // nibble k: total length of the first k + 1 symbols (1..8)
};

// A lane's output buffer: 16 bytes being filled (lo, hi) and up to NB - 1 full 16-byte blocks waiting (the newest
// last), so that 16 NB consecutive bytes leave in NB back-to-back stores: a lane's blocks of one 128-byte line then
// reach the L2 together instead of at eight different times.  All indices are compile-time: the blocks stay in
// registers.
template <int NB>
struct ByteSink {
    uint64_t lo = 0, hi = 0;
    uint4 wait[NB - 1] = {};
    uint32_t fill = 0, pending = 0, stored = 0;

    // Appends the `count` low bytes of `nb` (its other bytes are zero).
    __device__ __forceinline__ void append(uint64_t nb, uint32_t count, uint8_t *out)
    {
        const uint32_t sh = (fill & 7u) * 8u;
        const uint64_t x = nb << sh;
        const uint64_t y = sh ? nb >> (64u - sh) : 0ull;
        uint64_t carry = 0;
        if (fill < 8u) {
            lo |= x;
            hi |= y;
        } else {
            hi |= x;
            carry = y;
        }
        fill += count;
        if (fill >= 16u) {
            const uint4 blk{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
            if (pending == NB - 1) {
                uint4 *dst = reinterpret_cast<uint4 *>(out + stored);
#pragma unroll
                for (int j = 0; j < NB - 1; ++j)
                    dst[j] = wait[j];
                dst[NB - 1] = blk;
                stored += 16u * NB;
                pending = 0;
            } else {
#pragma unroll
                for (int j = 0; j < NB - 2; ++j)
                    wait[j] = wait[j + 1];
                wait[NB - 2] = blk;
                ++pending;
            }
            lo = carry;
            hi = 0;
            fill -= 16u;
        }
    }

    // Writes what is left: the waiting blocks (the last `pending` entries of wait), then the bytes of the partly
    // filled one.
    __device__ __forceinline__ void flush(uint8_t *out)
    {
        uint4 *dst = reinterpret_cast<uint4 *>(out + stored);
#pragma unroll
        for (int j = 0; j < NB - 1; ++j) {
            const int first = NB - 1 - (int)pending;             // wait[first..NB-2] are valid
            if (j >= first)
                dst[j - first] = wait[j];
        }
        stored += 16u * pending;
        pending = 0;
        for (uint32_t i = 0; i < fill; ++i)
            out[stored + i] = (uint8_t)((i < 8u ? lo >> (8u * i) : hi >> (8u * (i - 8u))) & 0xffu);
    }
};

__global__ __launch_bounds__(kHuffmanDirectWG) void k_huffman_decode_direct(HuffmanDecodeParams P, HuffmanCode H)
{
    extern __shared__ __align__(16) uint32_t stage_rows[];      // one staging row per thread
    __shared__ __align__(16) MultiEntry multi[256];
    __shared__ uint8_t lut8[256];
    __shared__ uint32_t first[16], count[16], offset[16], sorted[16];
    const uint32_t tid = threadIdx.x;
    const uint32_t S = 1u << P.sync_shift;
    if (tid < 16u) {
        first[tid] = H.first[tid];
        count[tid] = H.count[tid];
        offset[tid] = H.offset[tid];
        sorted[tid] = H.sorted[tid];
    }
    __syncthreads();
    {
        // entry `tid` of both tables: canonical decoding of the eight bits, symbol after symbol
        const uint32_t p = tid;
        uint32_t used = 0, n = 0, lo = 0, hi = 0, single = 0, cum = 0;
        for (;;) {
            uint32_t entry = 0;
            for (uint32_t L = 1; used + L <= 8u && L <= H.maxlen; ++L) {
                const uint32_t idx = ((p >> (8u - used - L)) & ((1u << L) - 1u)) - first[L];
                if (idx < count[L]) {
                    entry = sorted[offset[L] + idx] | (L << 4);
                    break;
                }
            }
            if (!used)
                single = entry;                                  // the first codeword alone, sign not needed here
            const uint32_t sym = entry & 15u, L = entry >> 4;
            const uint32_t bits = L + (sym ? 1u : 0u);
            if (!L || used + bits > 8u)
                break;
            const uint32_t neg = sym ? (p >> (8u - used - bits)) & 1u : 0u;
            const uint32_t byte = sym | (neg << 7);
            if (n < 4u)
                lo |= byte << (8u * n);
            else
                hi |= byte << (8u * (n - 4u));
            used += bits;
            cum |= used << (4u * n);
            ++n;
        }
        multi[p] = MultiEntry{lo, hi, n, cum};
        lut8[p] = (uint8_t)single;
    }
    __syncthreads();

    const HuffmanStream &W = P.w[blockIdx.y];
    const uint64_t u = (uint64_t)blockIdx.x * kHuffmanDirectWG + tid;
    if (u >= P.nb * P.nseg)
        return;
    const uint64_t b = u / P.nseg;
    const uint32_t g = (uint32_t)(u - b * P.nseg);
    const uint32_t nbk = (uint32_t)min((uint64_t)P.bucket, P.d - b * P.bucket);
    const uint32_t c_lo = g << P.sync_shift;
    if (c_lo >= nbk)
        return;
    const uint32_t n = min(nbk, c_lo + S) - c_lo;
    const uint32_t cap = huffman_stage_cap(S), stride = huffman_stage_stride(S);
    uint32_t *srow = stage_rows + tid * stride;
    const uint64_t start = (W.bit_off[b] + 31ull) & ~31ull, end = W.bit_off[b + 1];
    const uint32_t len = end > start ? (uint32_t)(end - start) : 0u;
    const uint32_t *sg = W.sync + b * P.nsync;
    const uint32_t lo = g ? sg[g - 1u] : 0u;
    const uint32_t hi = g + 1u < P.nseg ? sg[g] : len;
    bool bad = lo > hi || hi > len;
    uint8_t *out = W.q + b * P.bucket + c_lo;                   // 16-byte aligned
    const uint32_t w0 = lo >> 5, nw = bad ? 0u : ((hi + 31u) >> 5) - w0;
    if (!bad && nw <= cap) {
        const uint32_t *src = W.words + (start >> 5) + w0;
        for (uint32_t j0 = 0; j0 < nw; j0 += 8u) {
            uint32_t t[8];
#pragma unroll
            for (uint32_t j = 0; j < 8u; ++j)
                t[j] = src[min(j0 + j, nw - 1u)];
#pragma unroll
            for (uint32_t j = 0; j < 8u; ++j)
                if (j0 + j < nw)
                    srow[1u + j0 + j] = t[j];
        }
        const uint32_t bit0 = lo & 31u;
        uint32_t p31 = bit0 + 31u, q = p31 >> 5;
        uint32_t hw = srow[q], lw = srow[q + 1u], nx = srow[q + 2u];
        ByteSink<4> sink;
        uint32_t i = 0;
        while (i < n) {
            const uint32_t w = __builtin_amdgcn_alignbit(hw, lw, ~p31);
            uint64_t nb;
            uint32_t cnt, bits;
            const uint4 e = *reinterpret_cast<const uint4 *>(&multi[w >> 24]);      // one 16-byte LDS read
            cnt = min(e.z, n - i);
            if (cnt) {
                bits = (e.w >> (4u * (cnt - 1u))) & 15u;
                const uint64_t keep = cnt == 8u ? ~0ull : (1ull << (8u * cnt)) - 1ull;
                nb = (((uint64_t)e.y << 32) | e.x) & keep;
            } else {
                uint32_t entry = lut8[w >> 24];
                if (!entry) {                                   // a codeword of nine bits or more (rare), or none
                    for (uint32_t L = 9; L <= H.maxlen; ++L) {
                        const uint32_t idx = (w >> (32u - L)) - first[L];
                        if (idx < count[L]) {
                            entry = sorted[offset[L] + idx] | (L << 4);
                            break;
                        }
                    }
                }
                const uint32_t sym = entry & 15u, L = entry >> 4;
                bad |= !L;
                const uint32_t neg = sym ? (w >> (31u - L)) & 1u : 0u;
                nb = sym | (neg << 7);
                cnt = 1u;
                bits = L + (sym ? 1u : 0u);
            }
            sink.append(nb, cnt, out);
            i += cnt;
            p31 += bits;
            const uint32_t qn = p31 >> 5;
            const bool moved = qn != q;
            hw = moved ? lw : hw;
            lw = moved ? nx : lw;
            q = qn;
            nx = srow[min(qn + 2u, stride - 1u)];
        }
        sink.flush(out);       // (a unit that is no multiple of 64: S = 32, or the vector's last bucket)
        bad |= lo - bit0 + (p31 - 31u) != hi;
    } else if (!bad) {                                          // a unit too long for its staging row
        WalkWords gw{W.words + (start >> 5)};
        BitReader<WalkWords> br;
        br.init(gw, lo, (len + 31u) >> 5);
        uint32_t pos = lo;
        for (uint32_t i = 0; i < n; ++i) {
            br.refill();
            const uint32_t w = br.peek();
            uint32_t entry = 0;
            for (uint32_t L = 1; L <= H.maxlen; ++L) {
                const uint32_t idx = (w >> (32u - L)) - first[L];
                if (idx < count[L]) {
                    entry = sorted[offset[L] + idx] | (L << 4);
                    break;
                }
            }
            const uint32_t sym = entry & 15u, L = entry >> 4;
            const uint32_t nb = L + (sym ? 1u : 0u);
            if (!L || pos + nb > hi) {
                bad = true;
                break;
            }
            const uint32_t neg = sym ? (w >> (31u - L)) & 1u : 0u;
            out[i] = (uint8_t)(sym | (neg << 7));
            br.skip(nb);
            pos += nb;
        }
        bad |= pos != hi;
    }
    if (bad)
        atomicOr(P.flags, kFlagMalformed);
}

// ------------------------------------------------- decode + average of K messages in one launch
// The tile decoder of the ERC path (decode_wave) with the parse of a Huffman-coded piece: piece g of a bucket is its
// coordinates [g * stride, (g + 1) * stride), bounded by the index entries g - 1 (0 for the first) and g.  The
// level|sign bytes are never written: a nonzero symbol's value goes straight into the tile's fp64 sum.
//
// With gradients nearly all symbols are level 0, and a canonical code gives the most frequent symbol the codeword
// "0" once it has one bit.  Then (zero_run) a step of the parse is one run of zero symbols = the window's leading
// zero bits, followed by one nonzero symbol when its codeword and sign still fit the 32-bit window: about as many
// steps as the ERC parse has records.  With any other code a step is one symbol.
struct HuffmanWaveCodec {
    static constexpr bool kDirect = false;
    static constexpr uint32_t kRowWords = 13, kFewWords = 11;      // gradient data: about ten words per piece of 256 coordinates; 13: eight workgroups per CU
    // LDS, 256 entries: symbol | length << 4 of the codeword the eight bits start with, 0 where that is "0" for symbol 0,
    // kNoCodeword where it has nine bits or more (the code is complete, the host has seen to that: every prefix is of some
    // codeword)
    static constexpr uint32_t kNoCodeword = 0x0fu;
    uint8_t *lut8;
    uint32_t *canon;        // LDS, 64 words: first[16], count[16], offset[16], sorted[16] of the canonical code
    const HuffmanCode *H;
    uint32_t s, sync_shift;
    struct Range {
        uint32_t bit_lo, bit_hi;    // from the bucket's first bit
        uint32_t c_lo, n;           // first coordinate (in the bucket) and number of coordinates
    };
    __device__ __forceinline__ void init(const DecodeParams &, uint32_t lane) const
    {
        if (lane < 16u) {
            canon[lane] = H->first[lane];
            canon[16u + lane] = H->count[lane];
            canon[32u + lane] = H->offset[lane];
            canon[48u + lane] = H->sorted[lane];
        }
        for (uint32_t p = lane; p < 256u; p += kWave) {
            uint32_t entry = kNoCodeword;
            for (uint32_t L = 1; L <= 8u && L <= H->maxlen; ++L) {
                const uint32_t idx = (p >> (8u - L)) - H->first[L];
                if (idx < H->count[L]) {
                    entry = H->sorted[H->offset[L] + idx] | (L << 4);
                    break;
                }
            }
            lut8[p] = (uint8_t)(entry == 0x10u ? 0u : entry);
        }
    }
    __device__ __forceinline__ void entries(const uint32_t *sy, uint32_t g, const DecodeParams &P, uint32_t &e_lo,
                                            uint32_t &e_hi) const
    {
        e_lo = g ? sy[min(g, P.nsync) - 1u] : 0u;
        e_hi = sy[min(g, P.nsync - 1u)];                              // (not looked at for the bucket's last piece)
    }
    __device__ __forceinline__ bool range(const DecodeParams &P, uint32_t g, uint32_t nbk, uint32_t e_lo, uint32_t e_hi,
                                          uint32_t len, Range &R, bool &bad) const
    {
        R.c_lo = g << sync_shift;
        if (R.c_lo >= nbk)
            return false;
        R.n = min(nbk - R.c_lo, 1u << sync_shift);
        R.bit_lo = e_lo & kSyncOffMask;
        R.bit_hi = g + 1u < P.nseg ? e_hi & kSyncOffMask : len;
        // (a coordinate costs at least one bit: a piece without bits, as of a message that was never received, is malformed)
        if (R.bit_lo >= R.bit_hi || R.bit_hi > len) {
            bad = true;
            return false;
        }
        return true;
    }
    // Two loops.  run_short, where no codeword is longer than eight bits (every code up to s = 7): with kRuns (symbol 0 is the
    // codeword "0") a step is a run of zeros and the symbol that ends it, if it does, else one symbol, of a bit or more; counts
    // and index in the form of the ERC parser (position counting down, level added to the exponent, the add of a step under the
    // next one's table read; with kRuns about 30 vector instructions where run_any has 40 and as many scalar ones).  Encode +
    // decode of 8 x 25.6 M coordinates at s = 3 264 -> 252 us, of 3 x 16.8 M at s = 5 218 -> 186; without kRuns, s = 7, of 8 x
    // 25.6 M 807 -> 708, of 3 x 16.8 M in buckets of 4096 352 -> 262, of 4 x 16.8 M in buckets of 512 424 -> 353.  run_any, one
    // symbol per step or a zero run with a codeword from the canonical tables, for codes with longer words.
    struct Parser {
        const uint8_t *lut8;
        const uint32_t *canon;
        TileSink sink;
        double wnorm;
        uint32_t maxlen;
        bool zero_run;              // symbol 0 is the codeword "0"
        int n, end;                 // ~(bits from the row's first word + 31)
        uint32_t hi, lo, nx;
        uint32_t i, count, c_lo;    // coordinates done, of how many, the first one's index
        template <class Words>
        __device__ __forceinline__ void load(const Words &words)
        {
            const uint32_t q = ~(uint32_t)n >> 5;
            hi = words.at(q);
            lo = words.at(q + 1u);
            nx = words.at(q + 2u);
        }
        template <class Words>
        __device__ __forceinline__ void run(const Words &words, int stop)
        {
            if (maxlen > 8u)
                run_any(words, stop);
            else if (zero_run)
                run_short<true>(words, stop);
            else
                run_short<false>(words, stop);
        }
        template <bool kRuns, class Words>
        __device__ __forceinline__ void run_short(const Words &words, int stop)
        {
            // zeros of a step: what is left of the piece's bits, and with a codeword and its sign 32 bits at most
            const uint32_t cap = 31u - maxlen;
            const uint64_t wbits = (uint64_t)__double_as_longlong(wnorm) & 0x7fffffffffffffffull;
            const uint32_t whi = (uint32_t)(wbits >> 32), wlo = (uint32_t)wbits;
            const uint32_t binade = whi - 0x00100000u < 0x7fe00000u ? 0x00100000u : 0u;
            const uint32_t origin = sink.place(c_lo), last = count - 1u;
            int m = n >> 5;
            uint32_t sym = 0, sign = 0, at = 0;         // of the step before: symbol, its sign bit on top, its place
            auto add_value = [&]() {
                if (sym) {
                    uint32_t mh = __umul24(sym, binade) + whi;
                    mh |= sign & 0x80000000u;
                    sink.add(at, __longlong_as_double((long long)(((uint64_t)mh << 32) | wlo)));
                }
            };
            while (n > stop) {
                const uint32_t w = __builtin_amdgcn_alignbit(hi, lo, (uint32_t)n);
                const uint32_t left = (uint32_t)(n - end);                         // bits, >= 1
                uint32_t zc = 0;
                if constexpr (kRuns) {
                    uint32_t z;                                                    // all ones for an all-zero window
                    asm("v_ffbh_u32 %0, %1" : "=v"(z) : "v"(w));
                    zc = min(min(z, left), cap);
                }
                const uint32_t w2 = w << zc;
                uint32_t e = lut8[w2 >> 24];                                       // 0 for eight bits that start with a 0
                __builtin_amdgcn_sched_barrier(0);
                add_value();
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (kRuns)
                    e = left > zc ? e : 0u;
                sym = e & 15u;
                const uint32_t L = e >> 4;
                sign = w2 << L;
                const uint32_t is = i + zc;
                at = origin + (min(is, last) << TileSink::kUnit);
                const uint32_t one = min(sym, 1u);
                i = is + (kRuns ? one : 1u);
                n = n - (int)zc - (int)L - (int)one;
                const int mn = n >> 5;
                const bool moved = mn != m;
                hi = moved ? lo : hi;
                lo = moved ? nx : lo;
                m = mn;
                nx = words.after(mn);
            }
            add_value();
        }
        template <class Words>
        __device__ __forceinline__ void run_any(const Words &words, int stop)
        {
            const uint32_t zcap = zero_run ? 30u - maxlen : 0u;   // zeros + codeword + sign: 31 bits of the window at most
            uint32_t p31 = ~(uint32_t)n, q = p31 >> 5;
            const uint32_t stop31 = ~(uint32_t)stop;
            while (i < count && p31 < stop31) {
                const uint32_t w = __builtin_amdgcn_alignbit(hi, lo, ~p31);
                const uint32_t z = zero_run ? (uint32_t)__clz((int)w) : 0u;       // 32 for an all-zero window
                const uint32_t left = count - i;
                const bool symbol = z <= zcap && z < left;       // a symbol that is not part of the zero run follows
                const uint32_t zc = min(min(z, zcap), left);
                const uint32_t w2 = w << zc;
                uint32_t entry = lut8[w2 >> 24];
                if (symbol && entry == kNoCodeword) {              // a codeword of nine bits or more
                    for (uint32_t L = 9; L <= maxlen; ++L) {
                        const uint32_t idx = (w2 >> (32u - L)) - canon[L];
                        if (idx < canon[16u + L]) {
                            entry = canon[48u + canon[32u + L] + idx] | (L << 4);
                            break;
                        }
                    }
                }
                // everything below is straight-line: a step without a symbol adds nothing and moves on by its zeros
                const uint32_t sym = symbol ? entry & 15u : 0u, L = entry >> 4;
                const uint32_t bits = zc + (symbol ? L + (sym ? 1u : 0u) : 0u);
                const uint32_t at = sink.place(c_lo + i + zc);
                i += zc + (symbol ? 1u : 0u);
                p31 += bits;
                const uint32_t qn = p31 >> 5;
                const bool moved = qn != q;
                hi = moved ? lo : hi;
                lo = moved ? nx : lo;
                q = qn;
                nx = words.at(qn + 2u);
                if (sym) {
                    const double mag = ldexp(wnorm, (int)sym);
                    const uint32_t neg = (w2 << L) & 0x80000000u;
                    const uint64_t vb = (uint64_t)__double_as_longlong(mag) | ((uint64_t)neg << 32);
                    sink.add(at, __longlong_as_double((long long)vb));
                }
            }
            n = (int)~p31;
            // (the compiler would otherwise carry which of the two conditions ended the loop through every step, in scalar masks)
            asm("" : "+v"(i));
            if (i >= count && n != end) {                         // bits beyond the last coordinate: no further row is asked for
                i = count + 1u;
                n = end;
            }
        }
        __device__ __forceinline__ void finish(bool &bad) const { bad |= i != count || n != end; }
    };
    __device__ __forceinline__ Parser parser(float norm, const TileSink &sink) const
    {
        return Parser{lut8, canon, sink, (double)norm * ldexp(1.0, -1 - (int)s), H->maxlen, H->len[0] == 1u};
    }
    __device__ __forceinline__ void start(Parser &U, const StagedWords &words, const Range &R) const
    {
        U.n = (int)~((R.bit_lo & 31u) + 31u);
        U.end = (int)~(R.bit_hi - (R.bit_lo & ~31u) + 31u);
        U.i = 0;
        U.count = R.n;
        U.c_lo = R.c_lo;
        U.load(words);
    }
};

template <int UPDATE>
__global__ __launch_bounds__(kWaveWG, 2) void k_decode_wave_huffman(DecodeParams P, HuffmanCode H)
{
    __shared__ uint8_t lut8[256];
    __shared__ uint32_t canon[64];
    decode_wave<HuffmanWaveCodec, UPDATE, kTileCoords>(P, HuffmanWaveCodec{lut8, canon, &H, P.s, P.sync_shift});
}

// ------------------------------------------------------------------ average of level bytes
struct AverageParams {
    const float *norms[kMaxBatch];
    const uint8_t *q[kMaxBatch];
    float *out;
    uint64_t d;
    uint32_t K;
    uint32_t bucket;
    uint32_t s;
    uint32_t lut_tabs;      // k_average_levels16<true>: buckets a workgroup can touch (value tables per worker in LDS)
    float scale;
    int accumulate;
};

// out[i] = [out[i] +] scale * sum_k norms_k[bucket] * sign * 2^(level - 1 - s) from K arrays of level|sign bytes:
// fp64 sum in worker order, rounded to fp32 (a prior is added in fp32 after that).  VEC = 4 when buckets are multiples
// of four and everything is aligned, else 1.
template <int VEC>
__global__ __launch_bounds__(256) void k_average_levels(AverageParams P)
{
    const uint64_t i0 = ((uint64_t)blockIdx.x * 256u + threadIdx.x) * VEC;
    if (i0 >= P.d)
        return;
    const uint64_t bk = P.d <= 0xffffffffull ? (uint64_t)((uint32_t)i0 / P.bucket) : i0 / P.bucket;
    double sum[VEC];
#pragma unroll
    for (int c = 0; c < VEC; ++c)
        sum[c] = 0.0;
    for (uint32_t k = 0; k < P.K; ++k) {
        uint32_t bytes;
        if constexpr (VEC == 4) {
            if (i0 + 3u < P.d) {
                bytes = *reinterpret_cast<const uint32_t *>(P.q[k] + i0);
            } else {
                bytes = 0;
                for (uint32_t c = 0; c < 4u && i0 + c < P.d; ++c)
                    bytes |= (uint32_t)P.q[k][i0 + c] << (8u * c);
            }
        } else {
            bytes = P.q[k][i0];
        }
        if (!bytes)
            continue;
        const double nrm = (double)P.norms[k][bk];
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            const uint32_t byte = (bytes >> (8 * c)) & 0xffu, level = byte & 0x7fu;
            if (level) {
                const double val = ldexp(nrm, (int)level - 1 - (int)P.s);
                sum[c] += (byte & 0x80u) ? -val : val;
            }
        }
    }
    const double sc = (double)P.scale;
#pragma unroll
    for (int c = 0; c < VEC; ++c) {
        if (i0 + c < P.d) {
            const float r = (float)(sc * sum[c]);
            P.out[i0 + c] = P.accumulate ? P.out[i0 + c] + r : r;
        }
    }
}

// Buckets that are multiples of 16 coordinates, 16-byte aligned arrays: 16 coordinates per thread, one 16-byte load per
// worker, four 16-byte stores.
template <bool kLut>
__global__ __launch_bounds__(256) void k_average_levels16(AverageParams P)
{
    // kLut: the value of every byte, norm * sign * 2^(level - 1 - s) in fp64, tabulated once per (bucket the workgroup
    // touches, worker): 32 entries indexed by (sign, level), level <= 15.  A byte then costs an index, an LDS read and
    // an fp64 add instead of the exponent arithmetic.
    extern __shared__ __align__(16) double avg_lut[];           // [lut_tabs][K][32]
    const uint64_t wg0 = (uint64_t)blockIdx.x * 4096u;
    const uint64_t bk_first = P.d <= 0xffffffffull ? (uint64_t)((uint32_t)wg0 / P.bucket) : wg0 / P.bucket;
    if constexpr (kLut) {
        const uint64_t nb = (P.d + P.bucket - 1) / P.bucket;
        const uint32_t total = P.lut_tabs * P.K * 32u;
        for (uint32_t e = threadIdx.x; e < total; e += 256u) {
            const uint32_t idx = e & 31u, k = (e >> 5) % P.K, tab = (e >> 5) / P.K;
            const uint32_t level = idx & 15u;
            double val = 0.0;
            if (bk_first + tab < nb && level) {
                val = ldexp((double)P.norms[k][bk_first + tab], (int)level - 1 - (int)P.s);
                val = (idx & 16u) ? -val : val;
            }
            avg_lut[e] = val;
        }
        __syncthreads();
    }
    const uint64_t i0 = ((uint64_t)blockIdx.x * 256u + threadIdx.x) * 16u;
    if (i0 >= P.d)
        return;
    const uint64_t bk = P.d <= 0xffffffffull ? (uint64_t)((uint32_t)i0 / P.bucket) : i0 / P.bucket;
    const bool whole = i0 + 15u < P.d;
    const double *tab = avg_lut + (uint32_t)(bk - bk_first) * P.K * 32u;
    double sum[16];
#pragma unroll
    for (int c = 0; c < 16; ++c)
        sum[c] = 0.0;
    for (uint32_t k = 0; k < P.K; ++k) {
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        if (whole) {
            // read once: non-temporal (0.183 -> 0.175 ms for decode + average on the benchmark's default workload)
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(P.q[k] + i0));
            w[0] = t.x;
            w[1] = t.y;
            w[2] = t.z;
            w[3] = t.w;
        } else {
            for (uint32_t c = 0; i0 + c < P.d; ++c)
                w[c >> 2] |= (uint32_t)P.q[k][i0 + c] << (8u * (c & 3u));
        }
        if (!(w[0] | w[1] | w[2] | w[3]))
            continue;
        if constexpr (kLut) {
            const double *tk = tab + k * 32u;
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const uint32_t byte = (w[c >> 2] >> (8 * (c & 3))) & 0xffu;
                sum[c] += tk[((byte >> 3) & 16u) | (byte & 15u)];
            }
        } else {
            const double nrm = (double)P.norms[k][bk];
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const uint32_t byte = (w[c >> 2] >> (8 * (c & 3))) & 0xffu, level = byte & 0x7fu;
                if (level) {
                    const double val = ldexp(nrm, (int)level - 1 - (int)P.s);
                    sum[c] += (byte & 0x80u) ? -val : val;
                }
            }
        }
    }
    const double sc = (double)P.scale;
    float r[16];
#pragma unroll
    for (int c = 0; c < 16; ++c)
        r[c] = (float)(sc * sum[c]);
    if (whole) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float4 o{r[4 * v], r[4 * v + 1], r[4 * v + 2], r[4 * v + 3]};
            float4 *dst = reinterpret_cast<float4 *>(P.out + i0) + v;
            if (P.accumulate) {
                const float4 prev = *dst;
                o.x += prev.x;
                o.y += prev.y;
                o.z += prev.z;
                o.w += prev.w;
            }
            *dst = o;
        }
    } else {
        for (uint32_t c = 0; i0 + c < P.d; ++c)
            P.out[i0 + c] = P.accumulate ? P.out[i0 + c] + r[c] : r[c];
    }
}

}  // namespace nuq
