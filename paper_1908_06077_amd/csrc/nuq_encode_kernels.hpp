// Norms, quantizer and ENCODE kernels (Def. 1, App. A) -- one team of threads per bucket.
//
// Element layout inside a team: thread t, row i holds the four consecutive coordinates
// 4*(i*TEAM + t) .. +3 of its bucket, so every row is one fully coalesced 16-byte load per
// lane.  Level/sign bytes are exchanged through LDS so that in the coding phase thread t
// owns the contiguous coordinates [t*C, (t+1)*C), C = 4*ceil(n / (4*TEAM)) <= 64.
#pragma once
#include "nuq_device.hpp"

namespace nuq {

constexpr uint32_t kFlagCapacity = 1u, kFlagNonfinite = 2u, kFlagMalformed = 4u;

// Decoder index of an ERC message: a bucket is cut into blocks of 2^kSyncBlockShift coordinates and the records of a
// block into 2^pieces_shift pieces of equal count.  An entry = bit offset of the piece's first record (bits 0..20) |
// that record's index inside its block (bits 21..31).
constexpr uint32_t kSyncBlockShift = 11;
constexpr uint32_t kSyncOffMask = 0x1FFFFFu;

constexpr uint32_t kMaxBatch = 32;   // workers per launch

// Per-worker pointers of a batched launch (blockIdx.y selects the worker).
struct EncodeWorker {
    const float *v;        // fused / quantize / norms input
    const uint8_t *q_in;   // encode-from-bytes input
    uint8_t *q_out;        // quantize output
    const float *norms_in; // quantize input
    float *norms_out;      // norms / fused output
    uint32_t *sync;        // [nb * nsync]
    uint64_t *bit_off;     // [nb + 1]
    uint32_t *words;
    uint64_t words_cap;
    uint64_t seed;
};

struct EncodeBatch {
    EncodeWorker w[kMaxBatch];
};

struct EncodeParams {
    uint64_t d;
    uint64_t nb;
    uint32_t bucket;
    uint32_t s;
    uint32_t sync_shift;   // Huffman-coded messages: log2(sync stride), 0 = no index
    uint32_t nsync;        // index entries per bucket (0 = no index)
    uint32_t pieces_shift; // ERC messages: log2(pieces per block)
    uint32_t nblk;         // ERC messages: blocks per bucket = ceil(bucket / 2048)
    uint32_t slot_words;   // staging words per bucket
    uint32_t rows;         // ceil(bucket / (4*TEAM))
    uint32_t lds_words;    // LDS words per team (kernels that do not work theirs out)
    uint32_t rec_cap;      // nonzeros of a bucket whose indices fit the team's LDS list
    uint32_t out_cap;      // words of a bucket's bit string that fit the team's LDS buffer
    uint64_t nb_stride;    // nb rounded up to a multiple of 4: stride between workers in units
    uint32_t *units;       // [K * nb_stride] words of bit string per workgroup of the encoder, worker-major (see k_finish)
    uint32_t *staging;     // [K * nb * slot_words]
    uint32_t *flags;
    uint32_t norm_linf;    // level-table mode: 0 = Euclidean norm, 1 = maximum norm
    uint32_t stream;       // teams of less than a wave: full buckets of eight rows are loaded non-temporally too (load_rows)
};

template <int TEAM>
struct TeamGeom {
    static constexpr int kWG = TEAM <= kWave ? 256 : TEAM;     // (barriers inside a team of several waves: it is alone)
    static constexpr int kTeamsPerWG = kWG / TEAM;
};

// A 16-byte load from any 4-byte aligned address: the hardware does not ask for more, only the C++ types do.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 load4(const float *p)
{
    const f32x4_any r = *reinterpret_cast<const f32x4_any *>(p);
    return float4{r.x, r.y, r.z, r.w};
}

// The same for 16 bytes of a result that this kernel does not read again (the averaged gradient): measured on the
// decoder, 3 % on 8192-coordinate buckets of eight workers and 15 % on 16384-coordinate buckets of four.
__device__ __forceinline__ void store_once4(float4 *p, float4 v)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(f32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<f32x4 *>(p));
}

// Load the four coordinates of vector `vi` of a bucket of `nbk` coordinates starting at `vb`.
__device__ __forceinline__ float4 load_vec4(const float *vb, uint32_t vi, uint32_t nbk)
{
    const uint32_t e0 = 4u * vi;
    if (e0 + 3u < nbk)
        return load4(vb + e0);
    float4 r{0.0f, 0.0f, 0.0f, 0.0f};
    if (e0 < nbk) {
        r.x = vb[e0];
        r.y = e0 + 1u < nbk ? vb[e0 + 1u] : 0.0f;
        r.z = e0 + 2u < nbk ? vb[e0 + 2u] : 0.0f;
    }
    return r;
}

// A bucket's rows into registers.  Gradients are read once, so teams of a wave or more load them non-temporally: the
// stream then does not push the staged bit strings, lengths and messages, which the next kernel reads, out of the caches
// (172 -> 164 us on 8192-coordinate buckets, 3 % on 16384).  Smaller teams, whose loads are 256- or 512-byte pieces, do
// so for full buckets of eight rows per thread (`stream`, stream_loads).  wg_base: the workgroup's first bucket (uniform),
// lane_off: coordinates from there to the team's bucket.  The addresses of a full bucket are a uniform base per row (scalar
// registers; the empty asm keeps the compiler from folding the row into the lanes' 64-bit addresses, two instructions per row
// and lane) plus one 32-bit lane offset (in the global address space by type: behind the asm the compiler would have to assume
// a generic pointer).
typedef const __attribute__((address_space(1))) char *GlobalBytes;
typedef const __attribute__((address_space(1))) f32x4_any *GlobalFloat4;
template <int TEAM, int VPT>
__device__ __forceinline__ void load_rows(float4 (&x)[VPT], const float *wg_base, uint32_t lane_off, uint32_t nbk,
                                          uint32_t rows, uint32_t tid, bool stream)
{
    if (__all(nbk == (uint32_t)VPT * TEAM * 4u)) {       // full buckets that fill every row
        const uint32_t off = 4u * (lane_off + 4u * tid);                           // bytes, below 2^18
        auto load = [&](auto once) {
#pragma unroll
            for (int i = 0; i < VPT; ++i) {
                GlobalBytes row = (GlobalBytes)wg_base + i * (16 * TEAM);
                f32x4_any r;
                if constexpr (decltype(once)::value) {
                    asm("" : "+s"(row));        // (also keeps the two kinds of loads from being merged into the plain one)
                    r = __builtin_nontemporal_load((GlobalFloat4)(row + off));
                } else {
                    r = *(GlobalFloat4)(row + off);
                }
                x[i] = float4{r.x, r.y, r.z, r.w};
            }
        };
        if constexpr (TEAM >= 64) {
            load(std::true_type{});
        } else if constexpr (VPT == 8) {
            if (stream)
                load(std::true_type{});
            else
                load(std::false_type{});
        } else {
            load(std::false_type{});
        }
    } else if (__all(nbk >= 4u)) {
        // Buckets that do not fill every row (their size, or the vector's end): addresses clamped to the last four
        // coordinates, so that no load is predicated or branched around and all are under way together; what came from too
        // far down is then shifted out, rows beyond the bucket size are cleared.  Predicated, as it was, a row's load was
        // waited for before the next one was issued: encode of 4 x 16.8 M
        // coordinates in buckets of 1000 (half a wave each) 107 -> 82 us, of 700 96 -> 85.
        const uint32_t top = nbk - 4u;
        auto first = [&](int i) { return 4u * ((uint32_t)i * TEAM + tid); };
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            const GlobalFloat4 at = (GlobalFloat4)((GlobalBytes)wg_base + 4u * (lane_off + min(first(i), top)));
            f32x4_any r;
            if constexpr (TEAM >= 64)
                r = __builtin_nontemporal_load(at);
            else
                r = *at;
            x[i] = float4{r.x, r.y, r.z, r.w};
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            const uint32_t over = first(i) - min(first(i), top);
            if ((uint32_t)i >= rows) {
                x[i] = float4{0.0f, 0.0f, 0.0f, 0.0f};
            } else if (__any(over != 0u)) {
                const bool one = over & 1u, two = over & 2u, gone = over >= 4u;
                const float4 t = x[i];
                const float t0 = one ? t.y : t.x, t1 = one ? t.z : t.y, t2 = one ? t.w : t.z, t3 = one ? 0.0f : t.w;
                x[i].x = gone ? 0.0f : two ? t2 : t0;
                x[i].y = gone ? 0.0f : two ? t3 : t1;
                x[i].z = gone || two ? 0.0f : t2;
                x[i].w = gone || two ? 0.0f : t3;
            }
        }
    } else {                                             // a bucket of fewer than four coordinates, or none, in the wave
        const float *vb = wg_base + lane_off;
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            x[i] = float4{0.0f, 0.0f, 0.0f, 0.0f};
            if ((uint32_t)i < rows)
                x[i] = load_vec4(vb, (uint32_t)i * TEAM + tid, nbk);
        }
    }
}

// sqrt(t) in fp64, correctly rounded, for t in [2^-80, 2^100], where nothing can overflow or become subnormal: the
// hardware's reciprocal square root as the seed, one step of Goldschmidt's iteration for the pair (g, h) -> (sqrt t,
// 1 / (2 sqrt t)), then two corrections by the residual t - g^2, which an fma gives exactly (Markstein).
__device__ __forceinline__ double sqrt_mid(double t)
{
    const double y = __builtin_amdgcn_rsq(t);
    double g = t * y, h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    g = __builtin_fma(__builtin_fma(-g, g, t), h, g);
    return __builtin_fma(__builtin_fma(-g, g, t), h, g);
}

// Bucket norm from a per-row accessor.  fp32 partial sums (four accumulators per thread), fp64 across the team; if the
// fp32 result could have lost range (tiny or huge sums) the whole sum is redone in fp64.  Every thread of the team
// returns the same value.  A team of several waves leaves the fp64 part to its first wave (the others wait): done by
// every wave for itself, as it was, it was 1.5 of the encoder's 26 vector instructions per coordinate.
// lds: kNormParts x TEAM floats and scratch: 16 doubles of LDS (teams of several waves), free until the second barrier inside.
template <int TEAM, int VPT, class Row>
__device__ __forceinline__ float team_norm(Row row, float *lds, double *scratch)
{
    constexpr int kParts = kNormParts<TEAM>;
    float part[kParts];
#pragma unroll
    for (int h = 0; h < kParts; ++h) {
        float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll
        for (int i = h; i < VPT; i += kParts) {
            const float4 x = row(i);
            a0 = __builtin_fmaf(x.x, x.x, a0);
            a1 = __builtin_fmaf(x.y, x.y, a1);
            a2 = __builtin_fmaf(x.z, x.z, a2);
            a3 = __builtin_fmaf(x.w, x.w, a3);
        }
        part[h] = (a0 + a1) + (a2 + a3);
    }
    double tot;
    float norm;
    bool fine;
    if constexpr (TEAM > kWave) {
        const uint32_t tid = threadIdx.x % TEAM;
#pragma unroll
        for (int h = 0; h < kParts; ++h)
            lds[tid + h * TEAM] = part[h];
        __syncthreads();
        if (tid < (uint32_t)kWave) {
            tot = (double)lds[tid];
#pragma unroll
            for (int w = 1; w < kParts * TEAM / kWave; ++w)
                tot += (double)lds[tid + w * kWave];
            tot = wave_sum_f64(tot);
            fine = tot >= 0x1p-80 && tot <= 0x1p100;
            if (tid == 0)
                reinterpret_cast<float *>(scratch)[0] = fine ? (float)sqrt_mid(tot) : -1.0f;
        }
        __syncthreads();
        norm = uniform_f32(reinterpret_cast<const float *>(scratch)[0]);
        fine = norm >= 0.0f;
    } else {
        double p[kParts];
#pragma unroll
        for (int h = 0; h < kParts; ++h)
            p[h] = (double)part[h];
        tot = team_sum_f64<TEAM>(p, scratch);
        fine = tot >= 0x1p-80 && tot <= 0x1p100;
        norm = (float)sqrt_mid(tot);
    }
    if (!fine) {                 // (a NaN comes here too)
        double p[kParts];
#pragma unroll
        for (int h = 0; h < kParts; ++h) {
            p[h] = 0.0;
#pragma unroll
            for (int i = h; i < VPT; i += kParts) {
                const float4 x = row(i);
                p[h] += (double)x.x * (double)x.x;
                p[h] += (double)x.y * (double)x.y;
                p[h] += (double)x.z * (double)x.z;
                p[h] += (double)x.w * (double)x.w;
            }
        }
        norm = (float)sqrt(team_sum_f64<TEAM>(p, scratch));
    }
    return norm;
}

// ------------------------------------------------------------------ norms kernel
template <int TEAM, int VPT>
__global__ __launch_bounds__(TeamGeom<TEAM>::kWG) void k_bucket_norms(EncodeParams P, EncodeBatch Wk)
{
    __shared__ double scratch[16];
    __shared__ float part[TEAM > kWave ? kNormParts<TEAM> * TEAM : 1];
    const EncodeWorker &W = Wk.w[blockIdx.y];
    const uint32_t tid = threadIdx.x % TEAM;
    const uint64_t b = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG + threadIdx.x / TEAM;
    const bool active = b < P.nb;
    const uint64_t base = active ? b * P.bucket : 0;
    const uint32_t nbk = active ? (uint32_t)min((uint64_t)P.bucket, P.d - base) : 0u;
    const float *vb = W.v + base;
    auto row = [&](int i) { return load_vec4(vb, (uint32_t)i * TEAM + tid, nbk); };
    const float nrm = team_norm<TEAM, VPT>(row, part, scratch);
    if (active && tid == 0)
        W.norms_out[b] = nrm;
}

// Level of one coordinate (any magnitude) for the draw u: |v| is scaled into [ns, 2 ns) by replacing its exponent (its
// distance to the lower end of its bin, divided by the bin's width in units of c, is then a - ns for every bin), bin index
// from the difference of the bit patterns.  No branches.
__device__ __forceinline__ uint32_t quantize_any(float x, float u, const BucketScale &B)
{
    const int diff = (int)((f2u(x) & 0x7fffffffu) - B.ns_bits);
    const int m = diff >> 23;                          // bin: floor(log2(a / ns)), negative below the first level
    const float a2 = u2f(B.ns_bits + ((uint32_t)diff & 0x007fffffu));
    const float t = __builtin_fmaf(u, B.c, -(m < 0 ? fabsf(x) : a2 - B.ns));
    return (uint32_t)min(max(m, -1) + 1 + (t < 0.0f ? 1 : 0), B.s + 1);   // m >= s: the top level, no draw
}

// How a quantized coordinate is handed on, four to a word.  sg: four sign bytes (top bytes of the coordinates), tb: four
// bytes whose bit 7 says "not zero", tb2: four bytes whose bit 7 says "level 2", levels: four level indices.
//
// PlainBytes: level index | sign << 7, the byte of nuq_quantize (0 for a zero).
struct PlainBytes {
    __device__ __forceinline__ uint32_t first(uint32_t sg, uint32_t tb) const
    {
        const uint32_t up7 = tb & 0x80808080u;
        return (sg & up7) | (up7 >> 7);
    }
    __device__ __forceinline__ uint32_t two(uint32_t sg, uint32_t tb, uint32_t tb2) const
    {
        const uint32_t up7 = tb & 0x80808080u;
        return (sg & up7) | ((up7 >> 7) + ((tb2 >> 7) & 0x01010101u));
    }
    __device__ __forceinline__ uint32_t any(uint32_t sg, uint32_t levels) const
    {
        return (sg & ((levels + 0x7f7f7f7fu) & 0x80808080u)) | levels;
    }
};
// FlagBytes, for the coding phase: bit 6 = not zero; the other bits only mean something where it is set: level index - 1
// from bit 0, sign where sign_shift moves bit 7 to.  The nonzero mask is then one AND and one byte dot product per word.
struct FlagBytes {
    uint32_t sign_shift, sign_mask;
    __device__ __forceinline__ uint32_t first(uint32_t sg, uint32_t tb) const
    {
        return ((sg >> sign_shift) & sign_mask) | ((tb >> 1) & 0x40404040u);
    }
    __device__ __forceinline__ uint32_t two(uint32_t sg, uint32_t tb, uint32_t tb2) const
    {
        return first(sg, tb) | ((tb2 >> 7) & 0x01010101u);
    }
    __device__ __forceinline__ uint32_t any(uint32_t sg, uint32_t levels) const
    {
        return ((sg >> sign_shift) & sign_mask) | (levels + 0x3f3f3f3fu);
    }
};

// Quantize the four coordinates of one vector; returns the four bytes in format F.
// x0 = (k0 + index of first coordinate) * C1.  The caller has applied B.prescale to x.
//
// Three routes, chosen per wave from the largest |v_i| of the vector over all lanes:
//   below the first level (the usual case: |v_i| < 2^-s ||v||): the level is 0 or 1, "up" is the sign bit of
//     t = fma(u, c, -|v|), and the bytes are assembled from the top bytes of v (sign) and t (up) with byte permutes;
//   below twice the first level: bins [0, ns) and [ns, 2 ns) have the same width, and u c < ns, so the level is
//     the number of negative ones among t and t' = fma(u, c, ns - |v|): t is negative whenever |v| >= ns, t' never is
//     when |v| < ns (ns - |v| is exact where it decides).  Without the selection of a bin per coordinate: 2.5 of 17
//     instructions less;
//   anything else: quantize_any.
//
// kNaN: the coordinates may hold a NaN (a finite norm that the caller supplies need not see it; under the fused kernels'
// own norm such a bucket is empty).  It must not choose the route: fmaxf drops every NaN, max_abs4 a signaling one in three
// of its four places.  And its t and t' carry a sign bit each, which would be level 2 by the second route: ns - |v| is at
// most ns, so the minimum of the two only moves a NaN, and t' is then not negative.
template <bool kNaN = false, class F>
__device__ __forceinline__ uint32_t quantize_vec4(const float4 &x, uint32_t x0, uint32_t k1, const BucketScale &B,
                                                  const F &fmt)
{
    const float xs[4] = {x.x, x.y, x.z, x.w};   // already multiplied by B.prescale
    const float big = kNaN ? fmaxf(fmaxf(fabsf(xs[0]), fabsf(xs[1])), fmaxf(fabsf(xs[2]), fabsf(xs[3]))) : max_abs4(xs);
    float u[4], t[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
        u[c] = (float)draw24(x0 + (uint32_t)c * kRngC1, k1);
    if (__all(big < B.ns2)) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            t[c] = __builtin_fmaf(u[c], B.c, -fabsf(xs[c]));
        const uint32_t sg = top_bytes(xs), tb = top_bytes(t);
        if (__all(big < B.ns))
            return fmt.first(sg, tb);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float below = B.ns - fabsf(xs[c]);
            t[c] = __builtin_fmaf(u[c], B.c, kNaN ? fminf(below, B.ns) : below);
        }
        return fmt.two(sg, tb, top_bytes(t));
    }
    uint32_t levels = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        levels |= quantize_any(xs[c], u[c], B) << (8 * c);
    return fmt.any(top_bytes(xs), levels);
}

// --------------------------------------------------------------- quantize kernel
template <int TEAM, int VPT>
__global__ __launch_bounds__(TeamGeom<TEAM>::kWG) void k_quantize(EncodeParams P, EncodeBatch Wk)
{
    const EncodeWorker &W = Wk.w[blockIdx.y];
    const uint32_t tid = threadIdx.x % TEAM;
    const uint64_t b = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG + team_uniform_u32<TEAM>(threadIdx.x / TEAM);
    if (b >= P.nb)
        return;
    const uint64_t base = b * P.bucket;
    const uint32_t nbk = (uint32_t)min((uint64_t)P.bucket, P.d - base);
    const float *vb = W.v + base;
    uint8_t *qb = W.q_out + base;
    const bool qaligned = (reinterpret_cast<uintptr_t>(qb) & 3u) == 0;
    const BucketScale B = make_scale(team_uniform_f32<TEAM>(W.norms_in[b]), (int)P.s);
    const BucketKey key = bucket_key(W.seed, b);
#pragma unroll 1
    for (uint32_t i = 0; i < P.rows; ++i) {
        const uint32_t vi = i * TEAM + tid;
        const uint32_t e0 = 4u * vi;
        if (e0 >= nbk)
            break;
        float4 x = load_vec4(vb, vi, nbk);
        if (B.prescale != 1.0f) {
            x.x *= B.prescale;
            x.y *= B.prescale;
            x.z *= B.prescale;
            x.w *= B.prescale;
        }
        const uint32_t packed = B.dead ? 0u : quantize_vec4<true>(x, (key.k0 + e0) * kRngC1, key.k1, B, PlainBytes{});
        if (qaligned && e0 + 3u < nbk) {
            reinterpret_cast<uint32_t *>(qb)[vi] = packed;
        } else {
            for (uint32_t c = 0; c < 4u && e0 + c < nbk; ++c)
                qb[e0 + c] = (uint8_t)(packed >> (8 * c));
        }
    }
}

// ----------------------------------------------------------------- coding phase
//
// On entry the team's bytes (FlagBytes) are in LDS (qb32, bytes at or beyond the bucket's length say "zero") and a
// barrier has been passed.  Produces the bucket's bit string in LDS, copies it to the staging area, writes its index entries.
// Every thread of the workgroup must call it (it contains barriers).
//
// Steps: (1) every thread finds the nonzeros of its contiguous chunk and the team compacts their indices into `rec` (a
// prefix sum gives the ranks); (2) the records are dealt out evenly, a thread takes a contiguous run of them, looks up
// their codes and sums their lengths; a second prefix sum gives every run its bit offset; (3) the run's records, kept in
// registers, are OR-ed into the bit string.
//
// LDS bounds the number of buckets in flight on a CU, and a bucket's worst case (every coordinate nonzero at the longest
// level code) is four to ten times what gradients produce.  So the team's index list and bit-string buffer hold `rec_cap`
// nonzeros and `out_cap` words, sized for the usual case, and a bucket that exceeds one of them takes a slower way:
//   nonzeros fit, bits fit  : as above
//   nonzeros fit, bits don't: the same, but records are OR-ed into the (zeroed) staging slot in global memory (teams of several
//                             waves; the others' buffer holds the longest string of as many records as are listed)
//   nonzeros don't fit      : Unlisted
//
// What bounds the kernel is dependent chains with too few waves beside them, then vector issue: eight workgroups per CU instead of
// five took 4 x 1.56 G coordinates in buckets of 512 from 6.65 to 6.00 ms, a quantizer of fewer and cheaper instructions nothing
// (8 x 25.6 M in buckets of 8192 1.002 times as fast).

// ERC of N (Alg. 2): groups binary(N), binary(bits(N) - 1), ... while the value is at least 2, last computed first, one 0.
struct ErcWord {
    uint32_t code, len;
};
constexpr uint32_t bit_width_c(uint32_t x)
{
    uint32_t w = 0;
    while (x) {
        ++w;
        x >>= 1;
    }
    return w;
}
constexpr ErcWord erc_c(uint32_t N)
{
    uint32_t code = 0, len = 0;
    for (uint32_t g = N; g >= 2u; g = bit_width_c(g) - 1u) {
        code |= g << len;
        len += bit_width_c(g);
    }
    return ErcWord{code << 1, len + 1u};
}

// 512 words of code tables per workgroup, built at compile time and copied to LDS.
//
// Large teams (buckets above 2048, one coordinate in ten nonzero or fewer: gaps of any size): 256 entries by gap (code |
// length << 16; entry 0 is not used) and 256 by byte: sign and level code, | their length << 16.
// Small teams (a coordinate in four nonzero: gaps below 32 but for one in 10^4): the whole record, code | length << 27,
// by byte and gap: 5 bits of gap, 3 of level, sign where levels are at most 8 (s <= 7), else 4 bits of gap, 4 of level.
struct CodeTables {
    uint32_t large[512], small[2][512];
};
constexpr CodeTables make_code_tables()
{
    CodeTables t{};
    for (uint32_t i = 0; i < 256u; ++i) {
        const ErcWord g = erc_c(i ? i : 1u), l = erc_c((i & 15u) + 1u);
        t.large[i] = g.code | (g.len << 16);
        t.large[256u + i] = ((i >> 7) << l.len) | l.code | ((l.len + 1u) << 16);
    }
    for (uint32_t v = 0; v < 2u; ++v)
        for (uint32_t i = 0; i < 512u; ++i) {
            const uint32_t gbits = v ? 4u : 5u, lbits = v ? 4u : 3u;
            const uint32_t gap = i & ((1u << gbits) - 1u), x = i >> gbits;
            const ErcWord g = erc_c(gap ? gap : 1u), l = erc_c((x & ((1u << lbits) - 1u)) + 1u);
            const uint32_t tail = ((x >> lbits) << l.len) | l.code;
            t.small[v][i] = (g.code << (l.len + 1u)) | tail | ((g.len + l.len + 1u) << 27);
        }
    return t;
}
__device__ const CodeTables kCodeTables = make_code_tables();

template <int TEAM>
constexpr bool kSmallTeam = TEAM <= kWave;
constexpr uint32_t kUsualRecords = 12, kKeptRecords = 2 * kUsualRecords;     // per thread of a small team (code_small)

// The byte format of the coding phase for the level count s.
template <int TEAM>
__device__ __forceinline__ FlagBytes flag_bytes(uint32_t s)
{
    if constexpr (kSmallTeam<TEAM>)
        return s <= 7u ? FlagBytes{4u, 0x08080808u} : FlagBytes{3u, 0x10101010u};
    else
        return FlagBytes{0u, 0x80808080u};
}

// nuq_encode's bytes (level index, sign in bit 7) in that format.  A level above s + 1 is the caller's error; it is coded
// modulo 16 (a multiple of 16 as 1), so that a record is never longer than one of level 15 and a receiver with fewer levels
// sees a level that it does not have.  Where the format has three bits of level, levels 9 to 15 set bit 4 too, which
// SmallRecords<true> looks at.
template <int TEAM>
__device__ __forceinline__ uint32_t flag_caller_bytes(const FlagBytes &fmt, uint32_t s, uint32_t w)
{
    const bool three_bits = kSmallTeam<TEAM> && s <= 7u;
    uint32_t levels = w & 0x7f7f7f7fu, above = 0;
    if (__builtin_expect((w & (three_bits ? 0x78787878u : 0x70707070u)) != 0u, 0)) {
        const uint32_t nonzero = ((levels + 0x7f7f7f7fu) >> 7) & 0x01010101u;
        levels &= 0x0f0f0f0fu;
        levels |= nonzero & ~((levels + 0x7f7f7f7fu) >> 7);
        if (three_bits) {
            above = (levels & 0x08080808u) & ((levels & 0x07070707u) + 0x07070707u);       // 9 to 15
            levels -= above;
        }
    }
    return fmt.any(w, levels) | (above << 1);
}

// The tables' way into LDS, in two halves: requested before the gradient's loads, stored when those are under way (a wait
// for the tables before they are requested would start every workgroup with an idle round trip).
template <int TEAM>
struct TableCopy {
    static constexpr uint32_t kWG = TeamGeom<TEAM>::kWG, kPer = kWG < 256u ? 512u / kWG : 2u, kStep = 512u / kPer;
    uint32_t words[kPer] = {};
    __device__ __forceinline__ explicit TableCopy(uint32_t s)
    {
        const uint32_t *src = kSmallTeam<TEAM> ? kCodeTables.small[s <= 7u ? 0 : 1] : kCodeTables.large;
        if (kWG == kStep || threadIdx.x < kStep)
#pragma unroll
            for (uint32_t i = 0; i < kPer; ++i)
                words[i] = src[threadIdx.x + i * kStep];
    }
    __device__ __forceinline__ void store(uint32_t *tables) const
    {
        if (kWG == kStep || threadIdx.x < kStep)
#pragma unroll
            for (uint32_t i = 0; i < kPer; ++i)
                tables[threadIdx.x + i * kStep] = words[i];
    }
};

// A record's bits (right-aligned) and length from its gap and byte.
struct LargeRecords {
    const uint32_t *tables;
    __device__ __forceinline__ uint32_t operator()(uint32_t gap, uint32_t byte, uint32_t &len) const
    {
        uint32_t lg, cg;
        if (gap < 256u) {
            const uint32_t e = tables[gap];
            lg = e >> 16;
            cg = e & 0xffffu;
        } else {
            cg = erc_code(gap, lg);
        }
        const uint32_t tl = tables[256u + byte];
        len = lg + (tl >> 16);
        return (cg << (tl >> 16)) | (tl & 0xffffu);
    }
};
// In one word (code | length << 27): a bucket of a small team has at most 2048 coordinates, so a record at most
// 19 + 1 + 7 = 27 bits (the last of 2048 coordinates alone, at level 15): exactly what the word has room for.
static_assert(erc_c(2048u).len + 1u + erc_c(15u).len <= 27u, "a small team's record beside its length in 32 bits");
// kCaller: the bytes are flag_caller_bytes'.
template <bool kCaller>
struct SmallRecords {
    const uint32_t *at;      // the table's entry for byte 0 (the "not zero" bit, 64, is part of every byte looked up)
    uint32_t gap_bits;       // 5 (levels up to 8) or 4
    __device__ __forceinline__ uint32_t packed(uint32_t gap, uint32_t byte) const
    {
        const uint32_t above = kCaller ? byte & (gap_bits == 5u ? 0x10u : 0u) : 0u;      // levels 9 to 15 beside 3 bits
        if (__builtin_expect((gap | (above << 1)) < (1u << gap_bits), 1))
            return at[(byte << gap_bits) | gap];
        const uint32_t lbits = 8u - gap_bits, x = (byte & 0x1fu) ^ above;
        uint32_t lg, ll;
        const uint32_t cg = erc_code(gap, lg), cl = erc_code((x & ((1u << lbits) - 1u)) + (above >> 1) + 1u, ll);
        return (((cg << 1) | (x >> lbits)) << ll) | cl | ((lg + ll + 1u) << 27);
    }
    __device__ __forceinline__ uint32_t operator()(uint32_t gap, uint32_t byte, uint32_t &len) const
    {
        const uint32_t r = packed(gap, byte);
        len = r >> 27;
        return r & 0x7ffffffu;
    }
};
template <int TEAM, bool kCaller>
__device__ __forceinline__ auto make_records(const uint32_t *tables, uint32_t s)
{
    if constexpr (kSmallTeam<TEAM>)
        return SmallRecords<kCaller>{tables - (s <= 7u ? 64 << 5 : 64 << 4), s <= 7u ? 5u : 4u};
    else
        return LargeRecords{tables};
}

// A thread's records, consecutive in the bit string, are shifted into a 64-bit register and leave it 32 bits at a time (a
// record is at most 31 bits, so at most 31 + 31 bits are pending), OR-ed into zeroed words because a thread's first and
// last word are shared with its neighbours.  Bits that have left stay in the register, above the pending ones, until they
// are shifted out: nothing reads them.  Words beyond `last` (modulo 2^32: those before dst too) are dropped.
struct BitWriter {
    uint32_t wi, fill;
    uint64_t acc;
    __device__ __forceinline__ explicit BitWriter(uint32_t bit) : wi(bit >> 5), fill(bit & 31u), acc(0) {}
    __device__ __forceinline__ void put(uint32_t *dst, uint32_t bits, uint32_t len, uint32_t last = ~0u)
    {
        acc = (acc << len) | bits;
        fill += len;
        if (fill >= 32u) {
            fill -= 32u;
            if (wi <= last)
                atomicOr(&dst[wi], __builtin_amdgcn_alignbit((uint32_t)(acc >> 32), (uint32_t)acc, fill));
            ++wi;
        }
    }
    __device__ __forceinline__ void flush(uint32_t *dst, uint32_t last = ~0u)
    {
        if (fill && wi <= last)
            atomicOr(&dst[wi], (uint32_t)(acc << (32u - fill)));
    }
};

// Orders a team's LDS traffic between the phases of the coding pass.  A team of one wave needs no hardware barrier
// (its lanes run in lockstep and its LDS operations complete in order), only the wait and a fence for the
// compiler; the teams of a workgroup are independent of each other.
template <int TEAM>
__device__ __forceinline__ void team_barrier()
{
    if constexpr (TEAM > kWave) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
    }
}

// A team's LDS, in 32-bit words.
struct TeamLds {
    uint32_t *qb32;        // rows * TEAM: bytes (teams of a wave or less: then `out`)
    uint16_t *rec;         // rec_cap indices ...
    uint32_t *out;         // ... then out_cap words of bit string (large teams); 16-byte aligned
    uint32_t *sync_l;      // nsync (buckets that are not listed) ...
    uint32_t *run_off;     // ... or TEAM (large teams, listed buckets): bit offset of every thread's run
    uint32_t *blk;         // nblk + 1 (large teams): records before each block of the index
    uint32_t *scratch;     // 64 (large teams)
    const uint32_t *tables;
};

// Where the coding phase puts its results: pointers out of the kernel's arguments, fetched before the gradient is waited for.
// (Fetched where they are used, a scalar load each in the last dependent steps of a workgroup's life, they cost 2 to 3 % of 8 x
// 25.6 M coordinates in buckets of 8192.)
struct EncodeOut {
    uint32_t *unit;        // staging area of the workgroup's buckets
    uint32_t *unit_words;  // words of their strings together
    uint64_t *bit_off;
    uint32_t *sync;
};
template <int TEAM>
__device__ __forceinline__ EncodeOut encode_out(const EncodeParams &P, const EncodeWorker &W)
{
    const uint64_t first = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG;
    EncodeOut O{P.staging + ((uint64_t)blockIdx.y * P.nb + first) * P.slot_words,
                P.units + (uint64_t)blockIdx.y * P.nb_stride + blockIdx.x, W.bit_off, W.sync};
    asm volatile("" : "+s"(O.unit), "+s"(O.unit_words), "+s"(O.bit_off), "+s"(O.sync));
    return O;
}

// What a thread knows of its bucket after step (1).
struct Chunk {
    uint64_t nz;           // mask of its chunk's nonzeros
    uint32_t base;         // in-bucket index of the chunk's first coordinate
    uint32_t rank0;        // records before the chunk
    uint32_t nnz;          // records of the bucket
};

// The bit string from LDS to its place in the staging area, with 16-byte stores.  Teams of several waves: the slot and the
// LDS words behind the string up to a multiple of four are the bucket's own.  Others: the next bucket's string follows at once,
// so the last piece ends with the string and takes words again that another piece has too.
template <int TEAM>
__device__ __forceinline__ void store_bucket(uint32_t *slot, const uint32_t *out, uint32_t nwords, uint32_t tid)
{
    if constexpr (TeamGeom<TEAM>::kTeamsPerWG == 1) {
        for (uint32_t i = 4u * tid; i < nwords; i += 4u * TEAM)
            *reinterpret_cast<uint4 *>(slot + i) = *reinterpret_cast<const uint4 *>(out + i);
    } else if (nwords >= 4u) {
        typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
        for (uint32_t i = 4u * tid; i < nwords; i += 4u * TEAM) {
            const uint32_t at = min(i, nwords - 4u);
            *reinterpret_cast<u32x4_any *>(slot + at) = u32x4_any{out[at], out[at + 1u], out[at + 2u], out[at + 3u]};
        }
    } else if (tid < nwords) {
        slot[tid] = out[tid];
    }
}

// Where a bucket's string of `total` bits goes: the strings of a workgroup's buckets (a unit) stand in its first bucket's slot
// and on, each from the next word.  In two steps, each called by all threads of the workgroup: its words are announced as soon
// as they are known, the place is worked out when the string is complete, after a barrier of the workgroup; asked for before
// the string was assembled it kept every team waiting for the workgroup's slowest in the middle of its life (8 x 0.3 M
// coordinates in buckets of 1000 12.0 us, 11.6 so).  Leaves what k_finish needs to know: every bucket's bit length, in the place
// of its offset, and the words of all of them.
// Each in a slot of its own, as they were, 27 words in 128 at 512 coordinates, left half-written lines and k_finish a bisection
// over buckets for every four words: k_finish of 4 x 1.56 G coordinates 703 -> 560 us.
template <int TEAM>
using UnitWords = uint32_t[TeamGeom<TEAM>::kTeamsPerWG];       // in LDS
template <int TEAM>
__device__ __forceinline__ void announce_bucket(UnitWords<TEAM> &words, bool active, uint32_t total)
{
    if (threadIdx.x % TEAM == 0)
        words[threadIdx.x / TEAM] = active ? (total + 31u) >> 5 : 0u;
}
template <int TEAM>
__device__ __forceinline__ uint32_t *place_bucket(const UnitWords<TEAM> &words, const EncodeOut &O, bool active, uint64_t b,
                                                  uint32_t total)
{
    constexpr uint32_t N = TeamGeom<TEAM>::kTeamsPerWG;
    static_assert(N > 1u && N <= (uint32_t)kRow, "one row of lanes scans the word counts");
    const uint32_t team = threadIdx.x / TEAM, row = threadIdx.x & (kWave - 1u) & ~(uint32_t)(kRow - 1);
    uint32_t inc = words[threadIdx.x & (N - 1u)];
    inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x111, 0xf, 0xf, true);   // row_shr:1
    inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x112, 0xf, 0xf, true);   // row_shr:2
    if constexpr (N > 4u)
        inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x114, 0xf, 0xf, true);   // row_shr:4
    if constexpr (N > 8u)
        inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x118, 0xf, 0xf, true);   // row_shr:8
    // (the first N lanes of a row hold the sums; N < 16: those behind start from them)
    if (active && threadIdx.x % TEAM == 0)
        O.bit_off[b + 1] = total;
    if (threadIdx.x == N - 1u)
        *O.unit_words = inc;
    const uint32_t end = (uint32_t)__shfl((int)inc, (int)(row | team), kWave);
    return O.unit + (end - (active ? (total + 31u) >> 5 : 0u));
}

// The same for a workgroup of one bucket, whose slot is its unit.  The lengths are left at the end: a store ahead of the
// barriers of the coding phase would be waited for there.
__device__ __forceinline__ void report_length(const EncodeOut &O, uint64_t b, uint32_t total, uint32_t tid)
{
    if (tid == 0) {
        O.bit_off[b + 1] = total;
        *O.unit_words = (total + 31u) >> 5;
    }
}

// Slots have room for the longest string of levels up to s + 1.  Levels above that (nuq_encode's caller's error: kCaller) can
// make a longer one; such a bucket is refused as a whole, whatever its neighbours hold: one word of ones in place of its
// string, which no decoder takes (its level code does not end), index entries of 0, and the flag.
constexpr uint32_t kRefusedBits = 32u;
template <bool kCaller>
__device__ __forceinline__ bool refused(const EncodeParams &P, uint32_t total)
{
    return kCaller && __builtin_expect((total + 31u) >> 5 > P.slot_words, 0);
}
template <int TEAM>
__device__ __forceinline__ void refuse_bucket(const EncodeParams &P, const EncodeOut &O, uint64_t b, uint32_t *slot)
{
    const uint32_t tid = threadIdx.x % TEAM;
    for (uint32_t i = tid; i < P.nsync; i += TEAM)
        O.sync[b * P.nsync + i] = 0u;
    if (tid == 0) {
        slot[0] = ~0u;
        atomicOr(P.flags, kFlagMalformed);
    }
}

// Buckets with more nonzeros than the list holds: every thread codes the records of its own chunk, in two passes; the bit
// string is assembled over the list's and the buffer's words together (the two regions are adjacent: seven tenths of the
// worst case), that of a small team's bucket in the list's place, which has room for a slot's words.  A string that does not fit
// there takes a second window over the same words.  OR-ed into the slot in global memory, as it was, the atomics were the whole
// time: 4 x 8 M coordinates at 9 bits each, buckets of 3000 1103 -> 142 us, of 8192 540 -> 139, of 32768 605 -> 206.
template <int TEAM, bool kCaller>
struct Unlisted {
    const EncodeParams &P;
    const TeamLds &L;
    const Chunk &C;
    int before;             // index of the last nonzero ahead of the thread's chunk
    uint32_t bits;          // of the chunk's records

    template <class F>
    __device__ __forceinline__ void for_my_records(F &&f) const
    {
        const uint8_t *qbytes = reinterpret_cast<const uint8_t *>(L.qb32);
        const auto record = make_records<TEAM, kCaller>(L.tables, P.s);
        int p = before;
        uint64_t m = C.nz;
        while (m) {
            const int e = (int)C.base + __ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            uint32_t len;
            const uint32_t rbits = record((uint32_t)(e - p), (uint32_t)qbytes[e], len);
            f(e, rbits, len);
            p = e;
        }
    }
    __device__ __forceinline__ void count()
    {
        const int last = C.nz ? (int)C.base + 63 - __clzll((long long)C.nz) : -1;
        before = team_exclusive_max<TEAM>(last, -1, reinterpret_cast<int *>(L.scratch + 16));
        bits = 0;
        for_my_records([&](int, uint32_t, uint32_t len) { bits += len; });
    }
    __device__ __forceinline__ uint32_t *string() const { return reinterpret_cast<uint32_t *>(L.rec); }
    // off0: the chunk's first bit, total: of the bucket.  The string of a small team's bucket is left at string().
    __device__ __forceinline__ void emit(const EncodeOut &O, bool active, uint64_t b, uint32_t off0, uint32_t total,
                                         uint32_t *slot = nullptr) const
    {
        const uint32_t tid = threadIdx.x % TEAM;
        const uint32_t nwords = (total + 31u) >> 5;
        uint32_t *const obuf = string();
        const uint32_t cap = kSmallTeam<TEAM> ? ~0u : (uint32_t)(L.out - obuf) + P.out_cap;   // a multiple of four
        auto clear = [&](uint32_t n) {
            for (uint32_t i = 4u * tid; i < n; i += 4u * TEAM)
                *reinterpret_cast<uint4 *>(obuf + i) = uint4{0u, 0u, 0u, 0u};
        };
        clear(min(nwords, cap));
        // index entries: their record numbers go to LDS (bit 31: a block without records), an entry past the last record is
        // the bucket's length, and whoever emits such a record writes the entry
        uint32_t *const sg = O.sync + (active ? b : 0) * P.nsync;
        const uint32_t pmask = (1u << P.pieces_shift) - 1u;
        for (uint32_t i = tid; i < P.nsync; i += TEAM) {
            const uint32_t f = kSmallTeam<TEAM> ? 0u : L.blk[i >> P.pieces_shift];       // (a small bucket is one block)
            const uint32_t n = kSmallTeam<TEAM> ? C.nnz : L.blk[(i >> P.pieces_shift) + 1u] - f;
            const uint32_t r = f + (((i & pmask) * n) >> P.pieces_shift);
            if (r >= C.nnz && active)
                sg[i] = total;
            L.sync_l[i] = r | (n ? 0u : 0x80000000u);
        }
        team_barrier<TEAM>();
        auto emit_first = [&](uint32_t last_word) {
            uint32_t t = off0, rno = C.rank0, cur = 0, hi = P.nsync;
            while (cur < hi) {                       // first entry at or after this thread's first record (they are sorted)
                const uint32_t mid = (cur + hi) >> 1;
                if ((L.sync_l[mid] & 0x7fffffffu) < rno)
                    cur = mid + 1u;
                else
                    hi = mid;
            }
            BitWriter w(off0);
            for_my_records([&](int e, uint32_t rbits, uint32_t len) {
                while (cur < P.nsync) {
                    const uint32_t tg = L.sync_l[cur];
                    if ((tg & 0x7fffffffu) != rno)
                        break;
                    const uint32_t rel = (tg >> 31) ? 0u : (uint32_t)e - ((cur >> P.pieces_shift) << kSyncBlockShift);
                    if (active)
                        sg[cur] = t | (rel << 21);
                    ++cur;
                }
                ++rno;
                t += len;
                w.put(obuf, rbits, len, last_word);
            });
            if (C.nz)
                w.flush(obuf, last_word);
        };
        if constexpr (kSmallTeam<TEAM>) {
            emit_first(~0u);
        } else if (nwords <= cap) {                                                  // uniform over the team
            emit_first(~0u);
            team_barrier<TEAM>();
            if (active)
                store_bucket<TEAM>(slot, obuf, nwords, tid);
        } else {
            emit_first(cap - 1u);
            team_barrier<TEAM>();
            if (active)
                store_bucket<TEAM>(slot, obuf, cap, tid);
            for (uint32_t lo = cap; lo < nwords; lo += cap) {
                team_barrier<TEAM>();
                clear(min(nwords - lo, cap));
                team_barrier<TEAM>();
                if (C.nz && (off0 + bits + 31u) >> 5 > lo) {
                    BitWriter w(off0);
                    w.wi -= lo;
                    for_my_records([&](int, uint32_t rbits, uint32_t len) { w.put(obuf, rbits, len, cap - 1u); });
                    w.flush(obuf, cap - 1u);
                }
                team_barrier<TEAM>();
                if (active)
                    store_bucket<TEAM>(slot + lo, obuf, min(nwords - lo, cap), tid);
            }
        }
    }
};

// Steps (2) and (3), teams of several waves: two or three records per thread.  The records' table entries, four of them
// kept; the index entries are looked up from the entry's side (the run that holds the record starts at run_off[owner]; the
// lengths of the records before it in that run are looked up again).
template <int TEAM, bool kCaller>
__device__ __forceinline__ void code_listed_large(const EncodeParams &P, const EncodeOut &O, bool active, uint64_t b,
                                              const TeamLds &L, uint32_t nnz)
{
    uint32_t *const slot = O.unit;
    const uint32_t tid = threadIdx.x % TEAM;
    const uint8_t *qbytes = reinterpret_cast<const uint8_t *>(L.qb32);
    const LargeRecords record{L.tables};
    const uint32_t per = (nnz + TEAM - 1u) / TEAM;
    const uint32_t r0 = min(tid * per, nnz), r1 = min(r0 + per, nnz);
    constexpr uint32_t kKept = 4;
    uint32_t kept_bits[kKept], kept_len[kKept], bits = 0;
    int p = r0 ? (int)L.rec[r0 - 1u] : -1;
#pragma unroll
    for (uint32_t i = 0; i < kKept; ++i) {
        kept_len[i] = 0;
        kept_bits[i] = 0;
        if (r0 + i < r1) {
            const int e = (int)L.rec[r0 + i];
            kept_bits[i] = record((uint32_t)(e - p), (uint32_t)qbytes[e], kept_len[i]);
            bits += kept_len[i];
            p = e;
        }
    }
    const int p_kept = p;
    for (uint32_t r = r0 + kKept; r < r1; ++r) {
        const int e = (int)L.rec[r];
        uint32_t len;
        record((uint32_t)(e - p), (uint32_t)qbytes[e], len);
        bits += len;
        p = e;
    }
    uint32_t total;
    const uint32_t off0 = team_exclusive_sum<TEAM, false>(bits, L.scratch + 16, total);
    const uint32_t nwords = (total + 31u) >> 5;
    const bool in_lds = nwords <= P.out_cap;                     // uniform over the team (the buffer was cleared before)
    if (refused<kCaller>(P, total)) {                            // (so is this)
        refuse_bucket<TEAM>(P, O, b, slot);
        report_length(O, b, kRefusedBits, tid);
        return;
    }
    if (P.nsync)
        L.run_off[tid] = off0;
    if (!in_lds) {
        if (active) {
            for (uint32_t i = tid; i < nwords; i += TEAM)
                slot[i] = 0u;
            __threadfence();   // the zeros are in place before any record is OR-ed over them
        }
        team_barrier<TEAM>();
    }
    auto emit_all = [&](uint32_t *dst) {
        BitWriter w(off0);
#pragma unroll
        for (uint32_t i = 0; i < kKept; ++i)
            if (kept_len[i])
                w.put(dst, kept_bits[i], kept_len[i]);
        int q = p_kept;
        for (uint32_t r = r0 + kKept; r < r1; ++r) {
            const int e = (int)L.rec[r];
            uint32_t len;
            const uint32_t rb = record((uint32_t)(e - q), (uint32_t)qbytes[e], len);
            w.put(dst, rb, len);
            q = e;
        }
        if (r0 < r1)
            w.flush(dst);
    };
    if (in_lds)
        emit_all(L.out);
    else if (active)
        emit_all(slot);
    team_barrier<TEAM>();
    uint32_t *const sg = O.sync + (active ? b : 0) * P.nsync;
    const uint32_t pmask = (1u << P.pieces_shift) - 1u;
    for (uint32_t i = tid; i < P.nsync; i += TEAM) {
        const uint32_t t = i >> P.pieces_shift;
        const uint32_t f = L.blk[t], n = L.blk[t + 1u] - f;
        const uint32_t r = f + (((i & pmask) * n) >> P.pieces_shift);
        uint32_t entry = total;
        if (r < nnz) {
            const uint32_t owner = r / per;
            uint32_t q0 = owner * per, pos = L.run_off[owner];
            int q = q0 ? (int)L.rec[q0 - 1u] : -1;
            for (; q0 < r; ++q0) {
                const int e = (int)L.rec[q0];
                uint32_t len;
                record((uint32_t)(e - q), (uint32_t)qbytes[e], len);
                pos += len;
                q = e;
            }
            entry = pos | ((n ? (uint32_t)L.rec[r] - (t << kSyncBlockShift) : 0u) << 21);
        }
        if (active)
            sg[i] = entry;
    }
    if (active && in_lds)
        store_bucket<TEAM>(slot, L.out, nwords, tid);
    report_length(O, b, total, tid);
}

// Steps (2) and (3), teams of a wave or less: around ten records per thread, each looked up once and kept as one word.
// A bucket is one block of the index and has at most one entry per thread.  While records are emitted, a record's place in
// the index list takes its bit offset instead (the list's 16 bits hold it: at most 2048 records of 27 bits), so the thread
// of entry i reads its record's index before and its offset after.
// A wave may hold teams whose bucket is listed and others whose is not; they come together where the workgroup's strings are
// placed.
template <int TEAM, bool kCaller>
__device__ __forceinline__ void code_small(const EncodeParams &P, const EncodeOut &O, bool active, uint64_t b,
                                       const TeamLds &L, const Chunk &C, bool listed)
{
    const uint32_t tid = threadIdx.x % TEAM;
    const uint32_t nnz = C.nnz;
    const uint8_t *qbytes = reinterpret_cast<const uint8_t *>(L.qb32);
    const uint32_t per = (nnz + TEAM - 1u) / TEAM;
    const uint32_t r0 = min(tid * per, nnz), n = min(r0 + per, nnz) - r0;
    // The first twelve are what gradients have; twelve more are kept where some lane of the wave has them (looked up again
    // for the emission they cost twice); more there are not (team_rec_cap).
    uint32_t kept[kKeptRecords] = {}, bits = 0;
    uint16_t *const run = L.rec + r0;
    const bool many = __any(listed && n > kUsualRecords);
    __shared__ UnitWords<TEAM> unit_words;
    Unlisted<TEAM, kCaller> U{P, L, C, -1, 0u};
    if (listed) {
        const auto record = make_records<TEAM, kCaller>(L.tables, P.s);
        int p = r0 ? (int)run[-1] : -1;
        auto look_up = [&](uint32_t i) {
            if (i < n) {
                const int e = (int)run[i];
                kept[i] = record.packed((uint32_t)(e - p), (uint32_t)qbytes[e]);
                bits += kept[i] >> 27;
                p = e;
            }
        };
#pragma unroll
        for (uint32_t i = 0; i < kUsualRecords; ++i)
            look_up(i);
        if (many)
#pragma unroll
            for (uint32_t i = kUsualRecords; i < kKeptRecords; ++i)
                look_up(i);
    } else {
        U.count();
        bits = U.bits;
    }
    uint32_t total;
    const uint32_t off0 = team_exclusive_sum<TEAM>(bits, nullptr, total);
    const uint32_t nwords = (total + 31u) >> 5;
    const bool refuse = refused<kCaller>(P, total);              // uniform over the team
    const uint32_t sent = refuse ? kRefusedBits : total;
    announce_bucket<TEAM>(unit_words, active, sent);
    const bool entry = listed && tid < P.nsync && nnz;
    const uint32_t r_entry = (tid * nnz) >> P.pieces_shift;      // < nnz for an entry
    const uint32_t e_entry = entry ? (uint32_t)L.rec[r_entry] : 0u;
    if (refuse) {
    } else if (!listed) {
        U.emit(O, active, b, off0, total);
    } else {                                                     // (the bytes have been read to the end: their place is free)
        for (uint32_t i = 4u * tid; i < nwords; i += 4u * TEAM)
            *reinterpret_cast<uint4 *>(L.out + i) = uint4{0u, 0u, 0u, 0u};
        team_barrier<TEAM>();
        BitWriter w(off0);
        uint32_t t = off0;
        auto emit = [&](uint32_t i) {
            if (kept[i]) {
                run[i] = (uint16_t)t;
                const uint32_t len = kept[i] >> 27;
                t += len;
                w.put(L.out, kept[i] & 0x7ffffffu, len);
            }
        };
#pragma unroll
        for (uint32_t i = 0; i < kUsualRecords; ++i)
            emit(i);
        if (many)
#pragma unroll
            for (uint32_t i = kUsualRecords; i < kKeptRecords; ++i)
                emit(i);
        if (n)
            w.flush(L.out);
    }
    __syncthreads();
    uint32_t *const slot = place_bucket<TEAM>(unit_words, O, active, b, sent);
    if (!active)
        return;
    if (refuse) {
        refuse_bucket<TEAM>(P, O, b, slot);
        return;
    }
    if (listed && tid < P.nsync)
        O.sync[b * P.nsync + tid] = entry ? (uint32_t)L.rec[r_entry] | (e_entry << 21) : 0u;
    store_bucket<TEAM>(slot, listed ? L.out : U.string(), nwords, tid);
}

// kCaller: the bytes are flag_caller_bytes'.
template <int TEAM, int VPT, bool kCaller>
__device__ __forceinline__ void encode_from_lds(const EncodeParams &P, const EncodeOut &O, bool active, uint64_t b,
                                            const TeamLds &L)
{
    const uint32_t tid = threadIdx.x % TEAM;
    const uint32_t rows = P.rows;
    Chunk C;
    C.base = tid * rows * 4u;

    // (1) nonzero mask of this thread's chunk (rows <= VPT <= 16 words: two 32-bit halves), ranks, compaction.  The mask of
    // two words is the byte dot products of their flags with 1, 2, 4, 8 and 16, 32, 64, 128, shifted left by 6.
    static_assert(VPT % 2 == 0 && VPT <= 16, "the chunk's mask is 64 bits, made of two words at a time");
    uint32_t half[2] = {0, 0};
#pragma unroll
    for (int w = 0; w < VPT; w += 2) {
        if ((uint32_t)w < rows) {
            const uint32_t *q = L.qb32 + tid * rows + (uint32_t)w;
            uint32_t m = __builtin_amdgcn_udot4(q[0] & 0x40404040u, 0x08040201u, 0u, false);
            if ((uint32_t)w + 1u < rows)
                m = __builtin_amdgcn_udot4(q[1] & 0x40404040u, 0x80402010u, m, false);
            half[w / 8] |= (w % 8 == 0 ? m >> 6 : m << (4 * (w % 8) - 6));
        }
    }
    C.nz = ((uint64_t)half[1] << 32) | half[0];
    C.rank0 = team_exclusive_sum<TEAM, false>((uint32_t)(__popc(half[0]) + __popc(half[1])), L.scratch, C.nnz);
    const bool listed = C.nnz <= P.rec_cap;        // uniform over the team
    if (P.nsync && !kSmallTeam<TEAM>) {
        // blk[t] = records before block t of the decoder index: the thread whose chunk holds the block's first
        // coordinate counts its own nonzeros below it (every block starts inside exactly one chunk)
        constexpr uint32_t kBlock = 1u << kSyncBlockShift;
        const uint32_t c = (C.base + kBlock - 1u) & ~(kBlock - 1u);
        const uint32_t t = c >> kSyncBlockShift;
        if (c < C.base + rows * 4u && t < P.nblk) {
            const uint32_t sh = c - C.base;                                  // < 64
            const uint64_t below = sh ? C.nz & (~0ull >> (64u - sh)) : 0ull;
            L.blk[t] = C.rank0 + (uint32_t)__popcll((unsigned long long)below);
        }
        if (tid == 0)
            L.blk[P.nblk] = C.nnz;
    }
    if (listed) {
        uint16_t *r = L.rec + C.rank0;
        auto list = [&](uint32_t m, uint32_t at) {
            while (m) {
                *r++ = (uint16_t)(at + (uint32_t)__builtin_ctz(m));
                m &= m - 1u;
            }
        };
        list(half[0], C.base);
        if constexpr (VPT > 8)
            list(half[1], C.base + 32u);
        if constexpr (!kSmallTeam<TEAM>)
            for (uint32_t i = 4u * tid; i < P.out_cap; i += 4u * TEAM)
                *reinterpret_cast<uint4 *>(L.out + i) = uint4{0u, 0u, 0u, 0u};
    }
    team_barrier<TEAM>();
    if constexpr (kSmallTeam<TEAM>) {
        code_small<TEAM, kCaller>(P, O, active, b, L, C, listed);
    } else if (listed) {
        code_listed_large<TEAM, kCaller>(P, O, active, b, L, C.nnz);
    } else {
        Unlisted<TEAM, kCaller> U{P, L, C, -1, 0u};
        U.count();
        uint32_t total;
        const uint32_t off0 = team_exclusive_sum<TEAM>(U.bits, L.scratch + 32, total);
        const bool refuse = refused<kCaller>(P, total);
        if (refuse)
            refuse_bucket<TEAM>(P, O, b, O.unit);
        else
            U.emit(O, active, b, off0, total, O.unit);
        report_length(O, b, refuse ? kRefusedBits : total, threadIdx.x);
    }
}

// Words of a team's bit-string buffer, a multiple of four like the slot's.  Teams of several waves: a quarter of the worst case.
// Teams of a wave or less keep every record of a listed bucket in registers before the first bit is written, so the string takes
// the place of the bytes it was made from, and more than that where it can be longer, which it can from s = 7 on (nine bits to a
// coordinate): the longest string of as many records as there may be is eight bits each for sign and level, and less than
// 1.5 bits of gap code to a coordinate (ERC(2) takes 3 bits, ERC(4) 6, others less for what they skip).  (For longer ones than the
// bytes' place records went to the slot in global memory one by one: 4 x 12 M coordinates at s = 14 in buckets of 64 4.84 ms, of 256
// 1.83, of 600 1.62, where 0.17, 0.10 and 0.11 do.)
__host__ __device__ inline uint32_t team_out_cap(uint32_t slot_words, uint32_t bucket, uint32_t team)
{
    const uint32_t quarter = (slot_words / 4u + 3u) & ~3u;
    if (team > (uint32_t)kWave)
        return slot_words <= 256u ? slot_words : quarter > 256u ? quarter : 256u;
    const uint32_t records = bucket < team * kKeptRecords ? bucket : team * kKeptRecords;
    const uint32_t longest = ((records * 8u + bucket + bucket / 2u + 31u) / 32u + 3u) & ~3u;
    return slot_words < longest ? slot_words : longest;
}

// Offsets of a team's LDS regions (see TeamLds), in words; `words` in all, a multiple of 4.  The workgroup's code tables
// follow the last team.
struct TeamLdsMap {
    uint32_t rec, out, sync, blk, run_off, scratch, words;
};
__host__ __device__ inline TeamLdsMap team_lds_map(uint32_t slot_words, uint32_t rows, uint32_t team, uint32_t rec_cap,
                                                   uint32_t out_cap, uint32_t nsync, uint32_t nblk)
{
    // (a bucket of a small team whose nonzeros do not fit the list assembles its string, a slot's words at most, in its place)
    const bool small = team <= (uint32_t)kWave;
    const uint32_t list = (rec_cap + 1u) / 2u, dense = small ? slot_words : 0u, bytes = rows * team;
    TeamLdsMap m;
    m.rec = small && out_cap > bytes ? out_cap : bytes;
    const uint32_t behind = m.rec + (((list > dense ? list : dense) + 3u) & ~3u);
    m.out = small ? 0u : behind;
    m.sync = behind + (small ? 0u : out_cap);
    m.run_off = m.sync;
    m.blk = m.sync + (small || nsync > team ? nsync : team);
    m.scratch = (m.blk + nblk + 2u) & ~1u;                         // 8-byte aligned
    m.words = ((small ? m.blk : m.scratch + 64u) + 3u) & ~3u;      // small teams need neither block counts nor scratch
    return m;
}

// Front of the fused kernels: the bucket's coordinates into registers (v is read once), its norm (written to
// norms_out), the quantizer; put(i, word) takes the bytes (format F) of the thread's row i < P.rows (coordinates
// 4 * (i * TEAM + tid) .. + 3), rows in ascending order; issued() is called once the loads are under way.  lds:
// kNormParts x TEAM words per team (teams of several waves) that put may be the next to write.
template <int TEAM, int VPT, class F, class Put, class Issued>
__device__ __forceinline__ void front_quantize(const EncodeParams &P, const EncodeWorker &W, uint64_t b, bool active,
                                               uint64_t base, uint32_t nbk, uint32_t tid, uint32_t *lds,
                                               uint32_t *scratch, const F &fmt, Put put, Issued issued)
{
    float4 x[VPT];
    const uint64_t wg_base = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG * P.bucket;
    load_rows<TEAM, VPT>(x, W.v + wg_base, active ? (uint32_t)(base - wg_base) : 0u, nbk, P.rows, tid, P.stream != 0u);
    issued();
    auto row = [&](int i) { return x[i]; };
    const float nrm = team_uniform_f32<TEAM>(
        team_norm<TEAM, VPT>(row, reinterpret_cast<float *>(lds), reinterpret_cast<double *>(scratch + 32)));
    const bool finite = nrm < __builtin_huge_valf();   // false for NaN too
    if (active && tid == 0) {
        W.norms_out[b] = nrm;
        if (!finite)
            atomicOr(P.flags, kFlagNonfinite);
    }
    const BucketScale B = make_scale(nrm, (int)P.s);
    const BucketKey key = bucket_key(W.seed, b);
    if (B.prescale != 1.0f) {   // tiny norm: work on the bucket scaled by a power of two
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            x[i].x *= B.prescale;
            x[i].y *= B.prescale;
            x[i].z *= B.prescale;
            x[i].w *= B.prescale;
        }
    }
    const uint32_t x0 = (key.k0 + 4u * tid) * kRngC1;      // row i starts 4 * TEAM * i coordinates further on
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        if ((uint32_t)i < P.rows)
            put(i, B.dead ? 0u : quantize_vec4(x[i], x0 + (uint32_t)i * (4u * TEAM * kRngC1), key.k1, B, fmt));
    }
}

// The same with the bytes into the team's LDS words qb32[rows * TEAM].
template <int TEAM, int VPT, class F, class Issued>
__device__ __forceinline__ void front_quantize_to_lds(const EncodeParams &P, const EncodeWorker &W, uint64_t b,
                                                      bool active, uint64_t base, uint32_t nbk, uint32_t tid,
                                                      uint32_t *qb32, uint32_t *scratch, const F &fmt,
                                                      Issued issued)
{
    front_quantize<TEAM, VPT>(P, W, b, active, base, nbk, tid, qb32, scratch, fmt,
                              [&](int i, uint32_t word) { qb32[(uint32_t)i * TEAM + tid] = word; }, issued);
}

// Front of the kernels that start from level|sign bytes: put(i, word) as for front_quantize, the bytes from q_in.
template <int TEAM, int VPT, class Put>
__device__ __forceinline__ void front_bytes(const EncodeParams &P, const EncodeWorker &W, uint64_t base, uint32_t nbk,
                                            uint32_t tid, Put put)
{
    const uint8_t *qg = W.q_in + base;
    const bool aligned = (reinterpret_cast<uintptr_t>(qg) & 3u) == 0;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        if ((uint32_t)i >= P.rows)
            break;
        const uint32_t vi = (uint32_t)i * TEAM + tid;
        const uint32_t e0 = 4u * vi;
        uint32_t word = 0;
        if (aligned && e0 + 3u < nbk) {
            word = reinterpret_cast<const uint32_t *>(qg)[vi];
        } else {
            for (uint32_t c = 0; c < 4u; ++c)
                if (e0 + c < nbk)
                    word |= (uint32_t)qg[e0 + c] << (8u * c);
        }
        put(i, word);
    }
}

template <int TEAM, int VPT>
__device__ __forceinline__ void front_bytes_to_lds(const EncodeParams &P, const EncodeWorker &W, uint64_t base,
                                                   uint32_t nbk, uint32_t tid, uint32_t *qb32)
{
    front_bytes<TEAM, VPT>(P, W, base, nbk, tid,
                           [&](int i, uint32_t word) { qb32[(uint32_t)i * TEAM + tid] = word; });
}

// Front of the fused kernels for an arbitrary level table T and the norm P.norm_linf selects: as front_quantize, with
// quantize_table_vec4 on the bucket's bins (kept in LDS).  put may be called a second time for a row (a row decided
// again): the last call counts.
template <int TEAM, int VPT, class F, class Put, class Issued>
__device__ __forceinline__ void front_quantize_table(const EncodeParams &P, const EncodeWorker &W, const LevelTable &T,
                                                     uint64_t b, bool active, uint64_t base, uint32_t nbk,
                                                     uint32_t tid, uint32_t *lds, uint32_t *scratch, const F &fmt, Put put,
                                                     Issued issued)
{
    __shared__ TableBins bins_all[TeamGeom<TEAM>::kTeamsPerWG];
    TableBins &bins = bins_all[threadIdx.x / TEAM];
    const float *vb = W.v + base;
    float4 x[VPT];
    const uint64_t wg_base = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG * P.bucket;
    load_rows<TEAM, VPT>(x, W.v + wg_base, active ? (uint32_t)(base - wg_base) : 0u, nbk, P.rows, tid, P.stream != 0u);
    issued();
    float nrm;
    if (P.norm_linf) {
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            m = max(max(m, f2u(x[i].x) & 0x7fffffffu), f2u(x[i].y) & 0x7fffffffu);
            m = max(max(m, f2u(x[i].z) & 0x7fffffffu), f2u(x[i].w) & 0x7fffffffu);
        }
        nrm = u2f(team_max_u32<TEAM>(m, scratch));
    } else {
        auto row = [&](int i) { return x[i]; };
        nrm = team_norm<TEAM, VPT>(row, reinterpret_cast<float *>(lds), reinterpret_cast<double *>(scratch + 32));
    }
    nrm = team_uniform_f32<TEAM>(nrm);
    const bool finite = nrm < __builtin_huge_valf();   // false for NaN too
    if (active && tid == 0) {
        W.norms_out[b] = nrm;
        if (!finite)
            atomicOr(P.flags, kFlagNonfinite);
    }
    const bool dead = !(nrm > 0.0f) || !finite;
    if (tid < 16u)
        fill_table_bins(bins, T, nrm, P.s, tid);
    team_barrier<TEAM>();
    const BucketKey key = bucket_key(W.seed, b);
    const TableRule R = make_table_rule<TEAM>(bins, P.s, P.s <= (P.norm_linf ? 3u : 7u));
    const bool all_exact = !dead && bins.thr[0] == 0.0f;
    uint32_t redo = 0;                                     // rows to be decided again by the fp64 rule (none if dead)
    const uint32_t x0 = (key.k0 + 4u * tid) * kRngC1;      // row i starts 4 * TEAM * i coordinates further on
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        if ((uint32_t)i < P.rows) {
            bool again = false;
            uint32_t q = 0;
            if (!dead)
                q = quantize_table_vec4<TEAM>(x[i], x0 + (uint32_t)i * (4u * TEAM * kRngC1), key.k1, R, fmt, again);
            put(i, q);
            redo |= (again ? 1u : 0u) << i;
        }
    }
    if (__any(all_exact))
        redo = dead ? 0u : (1u << P.rows) - 1u;
    while (redo) {                             // uniform over the wave's live lanes; the coordinates are loaded again
        const int i = __builtin_ctz(redo);
        redo &= redo - 1u;
        const uint32_t vi = (uint32_t)i * TEAM + tid;
        const uint32_t q = quantize_table_vec4_exact(load_vec4(vb, vi, nbk), key.k0 + 4u * vi, key.k1,
                                                     bins.edge, bins.edge[1], P.s, fmt);
        put(i, q);
    }
}

template <int TEAM, int VPT, class F, class Issued>
__device__ __forceinline__ void front_quantize_table_to_lds(const EncodeParams &P, const EncodeWorker &W,
                                                            const LevelTable &T, uint64_t b, bool active, uint64_t base,
                                                            uint32_t nbk, uint32_t tid, uint32_t *qb32, uint32_t *scratch,
                                                            const F &fmt, Issued issued)
{
    front_quantize_table<TEAM, VPT>(P, W, T, b, active, base, nbk, tid, qb32, scratch, fmt,
                                    [&](int i, uint32_t word) { qb32[(uint32_t)i * TEAM + tid] = word; }, issued);
}

// MODE 0: fused norms + quantize + encode from v.  MODE 1: encode from level/sign bytes.  MODE 2: as 0 for the level
// table T and the norm P.norm_linf selects (T is ignored in the other modes).
// (Small teams: eight waves per SIMD, as many as their LDS allows.)
template <int TEAM, int VPT, int MODE>
__global__ __launch_bounds__(TeamGeom<TEAM>::kWG, kSmallTeam<TEAM> && MODE == 0 ? 8 : 1) void k_encode(EncodeParams P,
                                                                                                      EncodeBatch Wk,
                                                                                                      LevelTable T)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const EncodeWorker &W = Wk.w[blockIdx.y];
    const uint32_t tid = threadIdx.x % TEAM;
    const uint32_t team = team_uniform_u32<TEAM>(threadIdx.x / TEAM);   // a scalar unless a wave holds several teams
    const TeamLdsMap map = team_lds_map(P.slot_words, P.rows, TEAM, P.rec_cap, P.out_cap, P.nsync, P.nblk);
    uint32_t *const lds = smem + team * map.words;
    uint32_t *const tables = smem + TeamGeom<TEAM>::kTeamsPerWG * map.words;
    const TeamLds L{lds, reinterpret_cast<uint16_t *>(lds + map.rec), lds + map.out, lds + map.sync, lds + map.run_off,
                    lds + map.blk, lds + map.scratch, tables};
    const TableCopy<TEAM> copy(P.s);
    // (Bytes are loaded row after row, so in teams of a few waves, of which many share a CU, the fetch's wait counts at the
    // kernel's start: 30 M coordinates in buckets of 14400 26.7 us, fetched behind the bytes 26.2.)
    constexpr bool kFetchLate = MODE == 1 && !kSmallTeam<TEAM> && TEAM <= 256;
    EncodeOut O;
    if constexpr (!kFetchLate)
        O = encode_out<TEAM>(P, W);

    const uint64_t b = (uint64_t)blockIdx.x * TeamGeom<TEAM>::kTeamsPerWG + team;
    const bool active = b < P.nb;
    const uint64_t base = active ? b * P.bucket : 0;
    const uint32_t nbk = active ? (uint32_t)min((uint64_t)P.bucket, P.d - base) : 0u;

    const FlagBytes fmt = flag_bytes<TEAM>(P.s);
    auto loads_issued = [&] { copy.store(tables); };
    if constexpr (MODE == 2) {
        front_quantize_table_to_lds<TEAM, VPT>(P, W, T, b, active, base, nbk, tid, L.qb32, L.scratch, fmt, loads_issued);
    } else if constexpr (MODE == 0) {
        front_quantize_to_lds<TEAM, VPT>(P, W, b, active, base, nbk, tid, L.qb32, L.scratch, fmt, loads_issued);
    } else {
        loads_issued();
        front_bytes<TEAM, VPT>(P, W, base, nbk, tid, [&](int i, uint32_t w) {
            L.qb32[(uint32_t)i * TEAM + tid] = flag_caller_bytes<TEAM>(fmt, P.s, w);
        });
        if constexpr (kFetchLate)
            O = encode_out<TEAM>(P, W);
    }
    __syncthreads();
    encode_from_lds<TEAM, VPT, MODE == 1>(P, O, active, b, L);
}

// ------------------------------------------------- offsets and gather of the strings
//
// wc_b = ceil(len_b / 32) words per bucket; start word of bucket b = sum of wc over the worker's
// earlier buckets; bit_off[b+1] = 32 * start_b + len_b.  One "finish" kernel per batch: a
// workgroup owns FB consecutive buckets of one worker, sums the words before them, writes their offsets and copies their
// strings from the staging area to their place in `words`.
//
// The encoder leaves len_b in bit_off[b+1] and, per workgroup of its own (1, 4, 8 or 16 buckets: a unit), the words of its
// buckets in `units`: the words before a group are a sum over units, taken directly or, for more than 8192 units, from
// per-chunk prefix sums.

constexpr uint32_t kChunk = 1024;          // units per chunk of the two-level sum
constexpr uint64_t kDirectSumMax = 8192;   // up to this many units every workgroup sums directly

__device__ __forceinline__ uint64_t block_sum_u64(uint64_t x, uint64_t *scratch /* 4 */)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        x += __shfl_xor((unsigned long long)x, off, kWave);
    __syncthreads();
    if ((threadIdx.x & 63u) == 0)
        scratch[threadIdx.x >> 6] = x;
    __syncthreads();
    return scratch[0] + scratch[1] + scratch[2] + scratch[3];
}

// chunk_sums[k * (nchunks + 1) + c] = words of worker k's units [c*1024, (c+1)*1024).  kBits: the n values are bit lengths
// of buckets, not words.
template <bool kBits>
__global__ __launch_bounds__(256) void k_chunk_sums(const uint32_t *units, uint64_t n, uint64_t stride,
                                                    uint64_t nchunks, uint64_t *chunk_sums)
{
    __shared__ uint64_t scratch[4];
    const uint32_t *u = units + (uint64_t)blockIdx.y * stride;
    const uint64_t i0 = (uint64_t)blockIdx.x * kChunk;
    uint64_t s = 0;
    for (uint32_t k = threadIdx.x; k < kChunk; k += 256u)
        if (i0 + k < n)
            s += kBits ? (u[i0 + k] + 31u) >> 5 : u[i0 + k];
    s = block_sum_u64(s, scratch);
    if (threadIdx.x == 0)
        chunk_sums[(uint64_t)blockIdx.y * (nchunks + 1) + blockIdx.x] = s;
}

// One workgroup per worker: chunk_sums[c] <- sum of chunk_sums[0..c) (in place).
__global__ __launch_bounds__(256) void k_chunk_scan(uint64_t *chunk_sums, uint64_t nchunks)
{
    __shared__ uint64_t carry;
    __shared__ uint64_t wave_tot[4];
    uint64_t *cs = chunk_sums + (uint64_t)blockIdx.x * (nchunks + 1);
    if (threadIdx.x == 0)
        carry = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint64_t i0 = 0; i0 < nchunks; i0 += 256) {
        const uint64_t i = i0 + threadIdx.x;
        const uint64_t v = i < nchunks ? cs[i] : 0ull;
        uint64_t inc = v;
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t t = __shfl_up((unsigned long long)inc, off, 64);
            if (lane >= off)
                inc += t;
        }
        if (lane == 63)
            wave_tot[wave] = inc;
        __syncthreads();
        uint64_t before = carry;
        for (int w = 0; w < wave; ++w)
            before += wave_tot[w];
        if (i < nchunks)
            cs[i] = before + inc - v;
        __syncthreads();
        if (threadIdx.x == 255)
            carry = before + inc;
        __syncthreads();
    }
}

// grid (ceil(nb / (FB * groups)), K), FB = 4, 16 or 64 buckets per group, a multiple of the unit (2^unit_shift buckets).
// chunk_prefix == nullptr: sum the units before the group directly.
//
// What bounds it is latency: a chain of dependent loads (lengths, then the strings they locate, and the units before the
// group), each a round trip, in a kernel of a few microseconds.  So the lengths and the units are requested together, the
// strings as soon as the lengths are there (their place in the staging area does not depend on the sum), and everything moves
// in pieces of four words (a unit's last piece may be shorter; any 4-byte aligned address takes a 16-byte store), each
// found by one bisection.
// kUnits: units of several buckets (groups of four: one unit).  Their words are read from `units`, not worked out from the
// lengths by shuffles between the two scans, and what is needed only where the message is full stays a loop (unrolled, its LDS
// reads took 16 registers): at most 64 vector registers, hence eight waves per SIMD.  With 66 to 78 it took 6.8 us instead of
// 5.2 for 1 x 12 M coordinates in buckets of 1500, whose 8000 waves are more than seven per SIMD.
template <uint32_t FB, uint32_t WG, bool kUnits>
__global__ __launch_bounds__(WG) void k_finish(EncodeParams P, EncodeBatch Wk, const uint64_t *chunk_prefix,
                                                uint64_t nchunks, uint32_t groups, uint32_t shift)
{
    const uint32_t unit_shift = kUnits ? (FB == 4u ? 2u : shift) : 0u;
    static_assert(FB == 4 || FB == 16 || FB == 64, "one wave scans the group's word counts");
    static_assert(WG == 64 || WG == 256, "block_sum_u64 adds four waves");
    __shared__ uint64_t scratch[4];
    __shared__ uint32_t wstart[FB + 1];   // first word of each bucket, relative to the group's first
    __shared__ uint32_t pstart[FB + 1];   // first piece of each unit
    const uint32_t nunits = FB >> unit_shift;                     // per group
    const EncodeWorker &W = Wk.w[blockIdx.y];
    const uint32_t *__restrict__ units = P.units + (uint64_t)blockIdx.y * P.nb_stride;
    const uint32_t tid = threadIdx.x;
    auto load_len = [&](uint64_t b0) {
        return tid < FB && b0 + tid < P.nb ? (uint32_t)W.bit_off[b0 + tid + 1] : 0u;
    };
    auto load_unit = [&](uint64_t b0) {
        return kUnits && tid < nunits && b0 + ((uint64_t)tid << unit_shift) < P.nb ? units[(b0 >> unit_shift) + tid] : 0u;
    };

    // A workgroup takes `groups` consecutive groups of FB buckets: the words before its first bucket are summed once
    // (from the chunk's start), after that the running total carries over from group to group.
    uint64_t b_first = (uint64_t)blockIdx.x * groups * FB;
    uint32_t my_len = load_len(b_first), my_unit = load_unit(b_first);
    const uint64_t u_first = b_first >> unit_shift;
    uint64_t lo = 0, base = 0;
    if (chunk_prefix) {
        const uint64_t c = u_first / kChunk;
        lo = c * kChunk;
        base = chunk_prefix[(uint64_t)blockIdx.y * (nchunks + 1) + c];
    }
    uint32_t part = 0;     // < 2^32: at most 8192 units of at most 2^16 words are summed here
    {
        const uint4 *__restrict__ u4 = reinterpret_cast<const uint4 *>(units + lo);
        const uint32_t n = (uint32_t)(u_first - lo), n4 = n >> 2;
#pragma unroll 4
        for (uint32_t i = tid; i < n4; i += WG) {
            const uint4 v = u4[i];
            part += v.x + v.y + v.z + v.w;
        }
        if (tid < (n & 3u))
            part += units[lo + 4u * n4 + tid];
    }
    bool summed = false;

    for (uint32_t g = 0; g < groups && b_first < P.nb; ++g, b_first += FB) {
        if (tid < kWave) {                      // the first wave: inclusive scans of the word and piece counts
            const uint32_t words = (my_len + 31u) >> 5;
            const uint32_t wi = wave_inclusive_sum(words), pi = wave_inclusive_sum(((kUnits ? my_unit : words) + 3u) >> 2);
            if (tid < FB) {
                wstart[tid + 1] = wi;
                pstart[tid + 1] = pi;
            }
            if (tid == 0)
                wstart[0] = pstart[0] = 0;
        }
        __syncthreads();
        const uint32_t len = my_len;
        if (g + 1u < groups) {
            my_len = load_len(b_first + FB);
            my_unit = load_unit(b_first + FB);
        }
        const uint32_t total = pstart[FB];
        const uint32_t *__restrict__ staging = P.staging + ((uint64_t)blockIdx.y * P.nb + b_first) * P.slot_words;
        constexpr uint32_t kFlight = 4;         // pieces per thread under way at once
        for (uint32_t p0 = tid; !summed || p0 < total; p0 += kFlight * WG) {
            uint4 x[kFlight];
            uint32_t bkt[kFlight], at[kFlight];
#pragma unroll
            for (uint32_t q = 0; q < kFlight; ++q) {
                const uint32_t p = p0 + q * WG;
                uint32_t j = 0;
#pragma unroll
                for (uint32_t step = FB / 2; step >= 1; step >>= 1)
                    if (!kUnits || step < nunits)
                        j += (pstart[j + step] <= p) ? step : 0u;
                bkt[q] = j << unit_shift;
                at[q] = 4u * (p - pstart[j]);
                if (p < total)
                    x[q] = *reinterpret_cast<const uint4 *>(staging + (uint64_t)bkt[q] * P.slot_words + at[q]);
            }
            if (!summed) {                      // (once, with the first pieces under way)
                if constexpr (WG == 64u) {
                    uint64_t y = part;
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1)
                        y += __shfl_xor((unsigned long long)y, off, kWave);
                    base += y;
                } else {
                    base += block_sum_u64(part, scratch);
                }
                if constexpr (kUnits)
                    base = uniform_u64(base);
                summed = true;
            }
            // a bucket's words are written if all of them fit
            uint32_t fit = wstart[FB];
            if (kUnits && base + fit > W.words_cap) {
                fit = 0;
#pragma unroll 1
                for (uint32_t i = 1; i < FB && base + wstart[i] <= W.words_cap; ++i)
                    fit = wstart[i];
            }
#pragma unroll
            for (uint32_t q = 0; q < kFlight; ++q) {
                const uint32_t w = wstart[bkt[q]] + at[q];
                uint32_t end = wstart[bkt[q] + (1u << unit_shift)];
                bool put = p0 + q * WG < total;
                if constexpr (kUnits) {
                    end = min(end, fit);
                    put = put && w < end;
                } else {
                    put = put && base + end <= W.words_cap;
                }
                if (put) {
                    uint32_t *dst = W.words + base + w;
                    typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
                    if (w + 4u <= end) {
                        *reinterpret_cast<u32x4_any *>(dst) = u32x4_any{x[q].x, x[q].y, x[q].z, x[q].w};
                    } else {
                        dst[0] = x[q].x;
                        if (w + 1u < end)
                            dst[1] = x[q].y;
                        if (w + 2u < end)
                            dst[2] = x[q].z;
                    }
                }
            }
        }
        if (tid < FB && b_first + tid < P.nb) {
            W.bit_off[b_first + tid + 1] = 32ull * (base + wstart[tid]) + len;
            if (b_first + tid == 0)
                W.bit_off[0] = 0;
            if (base + wstart[tid + 1] > W.words_cap && len)
                atomicOr(P.flags, kFlagCapacity);
        }
        base += wstart[FB];
        __syncthreads();          // the group's starts are read to the end before the next group overwrites them
    }
}

}  // namespace nuq
