// C ABI of the NUQSGD compression path (see include/nuq.h): argument checks, launch
// geometry and workspace layout.  All arithmetic of the method lives in the kernels.
#include "../../include/nuq.h"
#include "../../include/nuq_bench.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>
#include <type_traits>
#include <vector>

#include "nuq_decode_kernels.hpp"
#include "nuq_device.hpp"
#include "nuq_encode_kernels.hpp"
#include "nuq_fixed_kernels.hpp"
#include "nuq_huffman_kernels.hpp"
#include "nuq_sgd_kernels.hpp"
#include "nuq_table_kernels.hpp"

// Workspace of nuq_quantize_encode_static, the entry point that allocates nothing: staging slots, bit lengths and
// partial sums of the encoder's kernels.  Each device that loads the library holds its own copy until the process
// ends.  In host code this name only stands for the symbol: the device address comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[NUQ_STATIC_WORKSPACE_BYTES];

namespace {

using namespace nuq;

// Address of `scratch` on the current device, looked up once per device (with that device current) and kept.
void *static_workspace_ptr()
{
    static std::mutex mu;
    static void *ptrs[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p)
            return nullptr;
        ptrs[dev] = p;
    }
    return ptrs[dev];
}

// Sticky error flags, one word per device (each device holds its own copy of the symbol).
__device__ uint32_t g_flags;

// Their address on the current device, looked up once per device and kept (a symbol does not move).
uint32_t *flags_ptr()
{
    static std::atomic<void *> ptrs[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0)
        return nullptr;
    void *p = dev < 64 ? ptrs[dev].load(std::memory_order_relaxed) : nullptr;
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_flags)) != hipSuccess)
            return nullptr;
        if (dev < 64)
            ptrs[dev].store(p, std::memory_order_relaxed);
    }
    return static_cast<uint32_t *>(p);
}

// ---- optional per-launch timing (benchmarks only) ----
struct Timing {
    std::vector<hipEvent_t> start, stop;
    std::vector<int32_t> entry;
    uint32_t cap = 0, used = 0;
} g_timing;

struct ScopedTiming {
    hipStream_t st;
    int slot = -1;
    ScopedTiming(int entry, hipStream_t s) : st(s)
    {
        if (g_timing.used < g_timing.cap) {
            slot = (int)g_timing.used++;
            g_timing.entry[slot] = entry;
            (void)hipEventRecord(g_timing.start[slot], st);
        }
    }
    ~ScopedTiming()
    {
        if (slot >= 0)
            (void)hipEventRecord(g_timing.stop[slot], st);
    }
};

uint32_t erc_len_host(uint32_t N)
{
    uint32_t len = 1;
    while (N > 1) {
        uint32_t w = 0;
        for (uint32_t x = N; x; x >>= 1)
            ++w;
        len += w;
        N = w - 1;
    }
    return len;
}

// A level table: s + 2 finite values, 0 = l_0 < l_1 < ... < l_{s+1} = 1.
bool valid_levels(const float *lev, uint32_t s)
{
    if (lev[0] != 0.0f || lev[s + 1] != 1.0f)
        return false;
    for (uint32_t j = 0; j <= s; ++j)
        if (!(lev[j] < lev[j + 1]))
            return false;
    return true;
}

bool valid_common(uint64_t d, uint32_t bucket, uint32_t s)
{
    return d >= 1 && bucket >= 1 && bucket <= NUQ_MAX_BUCKET && s >= 1 && s <= NUQ_MAX_S;
}

bool valid_sync(uint32_t sync_stride)
{
    return sync_stride == 0 ||
           (sync_stride >= 64 && sync_stride <= 1024 && (sync_stride & (sync_stride - 1)) == 0);
}

uint32_t log2u(uint32_t x)
{
    uint32_t l = 0;
    while ((1u << l) < x)
        ++l;
    return l;
}

// Decoder index of an ERC message: blocks of 2048 coordinates per bucket, and log2 of the pieces per block (the
// smallest power of two that is at least min(bucket, 2048) / sync_stride).
uint32_t sync_blocks(uint32_t bucket)
{
    return (bucket + (1u << kSyncBlockShift) - 1u) >> kSyncBlockShift;
}

uint32_t sync_pieces_shift(uint32_t bucket, uint32_t sync_stride)
{
    const uint32_t span = std::min(bucket, 1u << kSyncBlockShift);
    return log2u((span + sync_stride - 1u) / sync_stride);
}

uint32_t slot_words_for(uint32_t bucket, uint32_t s)
{
    const uint64_t bits = (uint64_t)bucket * (2u + erc_len_host(s + 1));
    return (uint32_t)(((bits + 31) / 32 + 3) & ~3ull);   // 16-byte multiple
}

struct Workspace {
    uint32_t *units;
    uint64_t *chunk_sums;
    uint32_t *staging;
    uint64_t bytes;
};

Workspace carve(void *base, uint32_t K, uint64_t nb, uint32_t slot_words)
{
    auto up = [](uint64_t x) { return (x + 255) & ~255ull; };
    const uint64_t nchunks = (nb + kChunk - 1) / kChunk;
    uint64_t off = 0;
    Workspace w;
    char *p = static_cast<char *>(base);
    w.units = reinterpret_cast<uint32_t *>(p + off);
    off += up((uint64_t)K * ((nb + 3) & ~3ull) * 4);
    w.chunk_sums = reinterpret_cast<uint64_t *>(p + off);
    off += up((uint64_t)K * (nchunks + 1) * 8);
    w.staging = reinterpret_cast<uint32_t *>(p + off);
    off += up((uint64_t)K * nb * slot_words * 4);
    w.bytes = off;
    return w;
}

// What a kernel does with what the quantizer yields: codes it (kErc: main scheme, kErcOther: level tables, or bytes that the
// caller gives; kHuffman), packs codes of a level table, or stores it (kStore; or has no quantizer).
enum class TeamUse { kErc, kErcOther, kHuffman, kPackTable, kStore };

// Team shape per bucket size: (threads per bucket, float4 rows per thread).  kNarrow: half the threads, twice the rows, where
// narrow_teams<kUse> may ask for that.  Both form the same partial sums of a norm (kNormParts).  Rows that no bucket of the
// size has are loaded too (load_rows), hence the shapes of 4, 6 and 12 rows: packing 2 x 24.6 M coordinates at 8 bits in
// buckets of 10 000 takes 42.2 us with 12 rows, 46.2 with 16.
template <TeamUse kUse, bool kNarrow, class F>
int dispatch_team_as(uint32_t bucket, F &&f)
{
    using std::integral_constant;
    constexpr bool kNarrow4096 = kNarrow && kUse != TeamUse::kStore, kNarrow32768 = kNarrow4096 && kUse != TeamUse::kPackTable;
    if (bucket <= 256)   // four buckets per wave
        return f(integral_constant<int, 16>{}, integral_constant<int, 4>{});
    if (bucket <= 512)
        return f(integral_constant<int, 16>{}, integral_constant<int, 8>{});
    if (bucket <= 1024) {
        if constexpr (kNarrow)
            return f(integral_constant<int, 32>{}, integral_constant<int, 8>{});
        else
            return f(integral_constant<int, 64>{}, integral_constant<int, 4>{});
    }
    if (bucket <= 2048)
        return f(integral_constant<int, 64>{}, integral_constant<int, 8>{});
    if (bucket <= 4096) {
        if constexpr (kNarrow4096)
            return f(integral_constant<int, 128>{}, integral_constant<int, 8>{});
        else
            return f(integral_constant<int, 256>{}, integral_constant<int, 4>{});
    }
    if (bucket <= 8192)
        return f(integral_constant<int, 256>{}, integral_constant<int, 8>{});
    if (bucket <= 12288)
        return f(integral_constant<int, 256>{}, integral_constant<int, 12>{});
    if (bucket <= 16384)
        return f(integral_constant<int, 256>{}, integral_constant<int, 16>{});
    if constexpr (kNarrow32768)
        return bucket <= 24576 ? f(integral_constant<int, 512>{}, integral_constant<int, 12>{})
                               : f(integral_constant<int, 512>{}, integral_constant<int, 16>{});
    else
        return bucket <= 24576 ? f(integral_constant<int, 1024>{}, integral_constant<int, 6>{})
                               : f(integral_constant<int, 1024>{}, integral_constant<int, 8>{});
}

template <TeamUse kUse, class F>
int dispatch_team(uint32_t bucket, bool narrow, F &&f)
{
    return narrow ? dispatch_team_as<kUse, true>(bucket, f) : dispatch_team_as<kUse, false>(bucket, f);
}

// Nonzeros to be expected in a bucket of Gaussian coordinates whose first level is l1 of the norm: a coordinate of |z| standard
// deviations is sent with probability min(1, |z| / z1), z1 of them being the first level.  (The largest |z| of 300 to 800 is
// 3.2.)
double expected_nonzeros(uint32_t bucket, double l1, bool linf)
{
    const double z1 = l1 * (linf ? 3.2 : std::sqrt((double)bucket));
    return bucket * (std::sqrt(2.0 / M_PI) / z1 * -std::expm1(-0.5 * z1 * z1) + std::erfc(z1 / M_SQRT2));
}

// Whether nb buckets of each of K workers take the narrow shapes.  A team's fixed work (norm reduction, scale, key, scans,
// barriers) costs the fused encoders as much as a thousand coordinates per wave, so with half the waves per bucket a full chip
// gets through more buckets; a chip that is not full waits for a single bucket instead, which then takes longer.  The line is a
// number of buckets (wide against narrow in turn on the same gradients, some 2500 calls of random sizes):
//   above 16384: as soon as there are more buckets than CUs (256).  2.1 M coordinates in 258 buckets 21.7 -> 17.5 us, 30 M in
//     1500 of them 72 -> 48; 0.4 M in 27 buckets at s = 7 26.0 with 1024 threads, 32.0 with 512.  Huffman: from 1024 buckets
//     up to 24576 coordinates (4.9 M 34.2 -> 30.8; 600 buckets 27 and 30), never above (14 M 58 and 64).
//   2049 to 4096: from 2048 buckets of sparse levels (3390 buckets 18.3 -> 16.5 us, 1644 of them 14.5 and 15.3), 4096 of dense
//     ones, 8192 with the maximum norm (4292 buckets, s = 6, 56 and 64); Huffman from 4096 (5118: 23.9 -> 22.8; 2152: 14.8 and
//     15.1); packing with a level table from 8192 (8808: 31.4 -> 28.4; 6264: 35.7 and 36.9).
//   513 to 1024: from 5120 buckets (8937 of 600 coordinates 18.6 -> 14.9 us, 5916 14.9 -> 13.0, 4222 of 513 15.4 and 17.4),
//     where half a wave's rows waste less of a bucket (up to 832 coordinates: 28 % on 131 k buckets of 513) or levels are
//     sparse (13 k of 1000 22.5 -> 20.4; dense, 95 k of 1024 at s = 5, 9 % slower), but not with many levels from a table or
//     from bytes (55 k of 600, s = 14, 79 and 87), nor with more nonzeros than half a wave lists, 768 (58 k of 832 at s = 7 123
//     and 101, 62 k of 780 at s = 10 159 and 111); Huffman of more than 832 from 8192 (11 k of 1000 21.5 -> 20.9; 6.2 k of 1024
//     6 % slower).  All others, memory-bound: up to 640 coordinates, five rows where a wave loads 768, from 8192 buckets (packing
//     at 4 or 8 bits 15 % less on 50 k and more), up to 832 from 32768 (56 k of 700 9 % less, 17 k of 800 2 % more).
// What these shapes cost where the chip is not full: nuq_quantize on 0.2 M coordinates in buckets of 1000 3.8 us with a wave, 6.0
// with half; nuq_encode on 0.6 M in buckets of 3000 at s = 14 18.3 and 27.9; nuq_encode_huffman on 0.2 M in buckets of 1024 15.8
// and 20.8.
// Sparse: with the Euclidean norm a coordinate is norm / sqrt(bucket) on average, and with a first level l1 of three times that
// or more about a quarter of the coordinates or less are nonzero.
template <TeamUse kUse>
bool narrow_teams(uint64_t nb, uint32_t K, uint32_t bucket, uint32_t s, bool linf = false, double l1 = 0.0)
{
    const uint64_t teams = nb * K;
    const bool sparse = !linf && l1 * l1 * bucket >= 9.0;
    if constexpr (kUse == TeamUse::kErc || kUse == TeamUse::kErcOther) {
        if (bucket <= 1024u) {
            const bool fit = bucket <= 32u * kKeptRecords || sparse ||
                             (bucket <= 832u && expected_nonzeros(bucket, l1, linf) + 24.0 <= 32.0 * kKeptRecords);
            return teams >= 5120u && fit && (kUse == TeamUse::kErc || s <= 5u);
        }
        if (bucket <= 4096u)
            return teams >= (sparse ? 2048u : linf ? 8192u : 4096u);
        return teams > 256u;
    } else if constexpr (kUse == TeamUse::kHuffman) {
        if (bucket <= 1024u)
            return teams >= (bucket <= 832u ? 5120u : 8192u);
        return bucket <= 4096u ? teams >= 4096u : bucket <= 24576u && teams >= 1024u;
    } else {
        if (bucket <= 1024u)
            return (bucket <= 640u && teams >= 8192u) || (bucket <= 832u && teams >= 32768u);
        return kUse == TeamUse::kPackTable && bucket <= 4096u && teams >= 8192u;
    }
}

// Whether teams of less than a wave load full buckets of eight rows per thread, that is of exactly 512, or of 1024 in the narrow
// shape, non-temporally (load_rows; others load from clamped addresses, where it brought nothing: buckets of 1000 30.7 and 31.4 us).
// Four workers, buckets of 512, 12 M coordinates 55.1 -> 51.4 us to encode and 117 -> 107 a step with momentum, whose parameters and
// strings stay in the last-level cache; packing them at 4 bits 61 -> 57; 20 M in buckets of 1024 a step 169 -> 157; 40 M in a step 303
// -> 279; one encode of 200 M 200 -> 194, of 800 M 787 -> 755, of 1024 759 -> 713.  Beyond 1 G coordinates in all it no longer helps,
// for a reason that no measurement here has shown (far more than any cache holds on either side): 1 x 1.5 G 1430 and 1456 us, 4 x 0.4
// G 1540 and 1566, 4 x 0.8 G 3129 and 3253, in buckets of 1024 1320 and 1331, 1430 and 1427, 2847 and 2880.  Gradients of up to
// 32 MB in all are found in the eight L2 caches where they have just been written or encoded before: 4 x 1.5 M in buckets of 512 15.1
// and 16.0, of 1024 14.6 and 15.5, a step 29.3 and 30.2; at 8 M coordinates an encode alone still gains with plain loads (17.3 and
// 17.8), a step, whose parameters go through these caches too, no longer (34.0 and 33.1), hence 7 M.  Beyond that one gradient
// encoded again and again, as the variance diagnostic does, takes the same either way (12 M in buckets of 512 131.3 and 133.3 us a
// draw, of 1024 116.7 and 115.6).
// (Buckets of 256: 4 x 5 M 32.9 and 33.8; 4 x 20 M, a step 207 and 213.)
uint32_t stream_loads(uint64_t d, uint32_t K)
{
    return d > 7'000'000u / K && d <= (1ull << 30) / K ? 1u : 0u;
}

// Nonzeros that the LDS list of a team of the encoders holds (k_encode<TEAM, ., MODE>; l1, linf: its first level and norm).
//
// Teams of several waves: a quarter of the bucket (about four times what a Gaussian gradient produces), at least 1024; but of
// buckets of 12289 to 16384 no more than what five of them leave room for on a CU, as many as there are registers for (4 x 134 M
// heavy-tailed coordinates in buckets of 16384, both directions 605 us with four, 578 with five): 4076 of 16384 up to s = 6, 3820
// above, a quarter up to some 15300.  With 3584 for all, buckets of 15000 and 16384 with 0.23 to 0.245 of their coordinates nonzero
// took 183 and 190 us instead of 166 and 161 (4 x 30 M).  Level tables keep to 3584: their records are longer, so that what more is
// listed overflows the string's buffer (0.23 nonzero, exponential levels at s = 7, both directions 334 us, with 4096 951).  Encoding
// bytes gains nothing from a fifth workgroup (30 M, a tenth nonzero, 34.8 and 34.9 us, 0.23 46 with a quarter, 56 with 3584).
//
// Teams of a wave or less: all of a bucket's coordinates up to 256, where eight workgroups, as many as there are waves for, share
// a CU all the same, and above 512, but no more than kKeptRecords per thread.  257 to 512: what eight workgroups leave room for
// (six with a level table, whose kernel has registers for no more), which is all of a bucket up to some 350 coordinates and 300
// of 512.  A bucket that exceeds that costs half as much again, and where some do and others don't their waves go both ways.  So
// where more than that are to be expected, but no more than kKeptRecords per thread, the list is as long as that, with seven
// workgroups per CU (five); where still more are, it would be exceeded anyway.  4 x 12 M coordinates, 37 nonzeros in 64 for all ->
// this: s = 4 in buckets of 300 127 -> 80 us, of 400 110 -> 74, of 512 75 -> 67; s = 5 in 450 122 -> 82; the whole list at s = 5 in
// 512, 373 nonzeros of which it holds 384, would take 119 instead of 112.  QSGDinf at s = 3 in 300, both directions 227 -> 186.
template <int TEAM, int MODE>
uint32_t team_rec_cap(const EncodeParams &P, double l1)
{
    constexpr uint32_t kKept = TEAM * kKeptRecords, kTeams = TeamGeom<TEAM>::kTeamsPerWG;
    const uint32_t bucket = P.bucket;
    // LDS is given out in pieces of 1280 bytes; the list's words, a multiple of four, are what is free of a team's, or what the
    // string of a small team's unlisted bucket needs in their place
    constexpr uint32_t kCU = 160u * 1024u, kPiece = 1280u, kTables = MODE == 2 ? (uint32_t)sizeof(TableBins) : 0u,
                       kStatic = kTeams * (kTables + (kTeams > 1u ? 4u : 0u));
    const TeamLdsMap none = team_lds_map(P.slot_words, P.rows, TEAM, 0, P.out_cap, P.nsync, P.nblk);
    const uint32_t string = TEAM > kWave ? 0u : none.sync - none.rec;
    auto room = [&](uint32_t groups) {
        const uint32_t words = (kCU / groups / kPiece * kPiece - kStatic - 512u * 4u) / (4u * kTeams) & ~3u;
        return 2u * std::max(string, words - (none.words - string));
    };
    if constexpr (TEAM > kWave) {
        const uint32_t quarter = std::max(bucket / 4u, 1024u);
        if (bucket <= 12288u || bucket > 16384u || MODE == 1)
            return quarter;
        return std::min(quarter, MODE == 2 ? 3584u : room(5u));
    }
    if (TEAM > 16 || bucket <= 256u)
        return std::min(kKept, bucket <= 1024u ? bucket : 1024u);
    constexpr uint32_t kGroups = MODE == 2 ? 6u : 8u;
    const uint32_t useful = std::min(kKept, bucket);
    const uint32_t usual = std::min(useful, room(kGroups)), most = std::min(useful, room(kGroups - 1u));
    const double mean = expected_nonzeros(bucket, l1, P.norm_linf), sd = std::sqrt(mean * (1.0 - mean / bucket));
    const bool beyond = mean + 3.0 * sd + (P.norm_linf ? bucket / 16u : 0u) > usual;
    return beyond && mean + 1.5 * sd <= most ? most : usual;
}

// float4 rows of a bucket per thread.  Their TEAM words each are where team_norm's partial sums go before the bytes do.
template <int TEAM>
uint32_t team_rows(uint32_t bucket)
{
    return std::max<uint32_t>(TEAM > kWave ? kNormParts<TEAM> : 1, (bucket + 4 * TEAM - 1) / (4 * TEAM));
}

int check_launch()
{
    return hipGetLastError() == hipSuccess ? NUQ_OK : NUQ_EHIP;
}

// Grid of a per-bucket kernel: x = workgroups over the buckets of one worker, y = worker.
template <int TEAM>
bool bucket_grid(uint64_t nb, uint32_t K, dim3 &grid)
{
    const uint64_t gx = (nb + TeamGeom<TEAM>::kTeamsPerWG - 1) / TeamGeom<TEAM>::kTeamsPerWG;
    if (gx > 0x7fffffffull)
        return false;
    grid = dim3((uint32_t)gx, K);
    return true;
}

// Offsets and gather: lengths and staged strings of K workers into their bit_off and words.
template <uint32_t FB, uint32_t WG>
int launch_finish_as(const EncodeParams &P, const EncodeBatch &Wk, uint32_t K, const uint64_t *prefix, uint64_t nchunks,
                     uint32_t groups, uint32_t unit_shift, hipStream_t st)
{
    const uint64_t span = (uint64_t)FB * groups;
    const dim3 grid((uint32_t)((P.nb + span - 1) / span), K);
    if (unit_shift)
        hipLaunchKernelGGL((k_finish<FB, WG, true>), grid, dim3(WG), 0, st, P, Wk, prefix, nchunks, groups, unit_shift);
    else if constexpr (FB <= 16)                 // (groups of 64 buckets are of small ones)
        hipLaunchKernelGGL((k_finish<FB, WG, false>), grid, dim3(WG), 0, st, P, Wk, prefix, nchunks, groups, 0u);
    return check_launch();
}

int launch_finish(const EncodeParams &P, const EncodeBatch &Wk, uint32_t K, const Workspace &w, bool narrow, hipStream_t st)
{
    // buckets per workgroup of the encoder
    uint32_t unit_shift = 0;
    (void)dispatch_team<TeamUse::kErc>(P.bucket, narrow, [&](auto team_c, auto) {
        unit_shift = log2u(TeamGeom<decltype(team_c)::value>::kTeamsPerWG);
        return (int)NUQ_OK;
    });
    const uint64_t units = (P.nb + (1ull << unit_shift) - 1) >> unit_shift;
    const uint64_t nchunks = (units + kChunk - 1) / kChunk;
    const uint64_t *prefix = nullptr;
    if (units > kDirectSumMax) {
        hipLaunchKernelGGL(k_chunk_sums<false>, dim3((uint32_t)nchunks, K), dim3(256), 0, st, w.units, units, P.nb_stride,
                           nchunks, w.chunk_sums);
        hipLaunchKernelGGL(k_chunk_scan, dim3(K), dim3(256), 0, st, w.chunk_sums, nchunks);
        prefix = w.chunk_sums;
    }
    // Buckets per workgroup: 4 where there are few buckets (1427 of 8192 coordinates: 11.2 us with 16, 4.2 with 4; 24960 of
    // them: 9.2 with 16, 13.6 with 4, whose sums over the units before cost more than the copy), but at least a unit; 64
    // small ones where that still gives a chip's worth of workgroups, so that there is something to copy.  Very many small
    // buckets: one wave per workgroup (four times the groups in flight) and up to eight groups each (the sum before the
    // first is paid once).
    const uint64_t small_groups = (P.nb + 63) / 64 * K;
    if (P.bucket <= 1024u && small_groups >= 2u * 16384u)
        return launch_finish_as<64, 64>(P, Wk, K, prefix, nchunks, (uint32_t)std::min<uint64_t>(8, small_groups / 16384),
                                        unit_shift, st);
    if (P.bucket <= 1024u && small_groups >= 1024u)
        return launch_finish_as<64, 256>(P, Wk, K, prefix, nchunks, 1, unit_shift, st);
    if (unit_shift <= 2u && P.nb * K < 16u * 1024u)
        return launch_finish_as<4, 256>(P, Wk, K, prefix, nchunks, 1, unit_shift, st);
    return launch_finish_as<16, 256>(P, Wk, K, prefix, nchunks,
                                     (uint32_t)std::min<uint64_t>(8, std::max<uint64_t>(1, (P.nb + 15) / 16 * K / 16384)),
                                     unit_shift, st);
}

// Sizes of k_encode<., ., MODE> for K workers' buckets (l1, linf: its first level and norm) into P, and what f(team, rows per
// thread, LDS map) makes of them.
template <int MODE, class F>
int with_encode_shape(EncodeParams &P, uint32_t K, uint64_t d, uint32_t bucket, uint32_t s, uint32_t sync_stride, double l1,
                      bool linf, bool &narrow, F &&f)
{
    constexpr TeamUse kUse = MODE == 0 ? TeamUse::kErc : TeamUse::kErcOther;
    P.d = d;
    P.nb = nuq_num_buckets(d, bucket);
    P.nb_stride = (P.nb + 3) & ~3ull;
    P.bucket = bucket;
    P.s = s;
    P.nsync = nuq_num_sync(bucket, sync_stride);
    P.pieces_shift = P.nsync ? sync_pieces_shift(bucket, sync_stride) : 0;
    P.nblk = sync_blocks(bucket);
    P.slot_words = slot_words_for(bucket, s);
    P.norm_linf = linf ? 1u : 0u;
    P.stream = stream_loads(d, K);
    narrow = narrow_teams<kUse>(P.nb, K, bucket, s, linf, l1);
    return dispatch_team<kUse>(bucket, narrow, [&](auto team_c, auto vpt_c) {
        constexpr int TEAM = decltype(team_c)::value;
        P.rows = team_rows<TEAM>(bucket);
        P.out_cap = team_out_cap(P.slot_words, bucket, TEAM);
        P.rec_cap = team_rec_cap<TEAM, MODE>(P, l1);
        return f(team_c, vpt_c, team_lds_map(P.slot_words, P.rows, TEAM, P.rec_cap, P.out_cap, P.nsync, P.nblk));
    });
}

// MODE 0: fused norms + quantize + ENCODE from v.  MODE 1: ENCODE from level/sign bytes.  MODE 2: as 0 with the
// level table `levels` (host memory, s + 2 values) and the norm `norm_kind` selects.
template <int MODE>
int encode_batch(uint32_t K, const EncodeBatch &Wk, uint64_t d, uint32_t bucket, uint32_t s, uint32_t sync_stride,
                 void *workspace, uint64_t workspace_bytes, nuq_stream_t stream, const float *levels = nullptr,
                 uint32_t norm_kind = NUQ_NORM_L2)
{
    if (K < 1 || K > kMaxBatch || !valid_common(d, bucket, s) || !valid_sync(sync_stride) || !workspace ||
        (reinterpret_cast<uintptr_t>(workspace) & 15u))
        return NUQ_EINVAL;
    LevelTable T{};
    if (MODE == 2) {
        if (!levels || !valid_levels(levels, s) || (norm_kind != NUQ_NORM_L2 && norm_kind != NUQ_NORM_LINF))
            return NUQ_EINVAL;
        for (uint32_t j = 0; j < s + 2u; ++j)
            T.lev[j] = levels[j];
    }
    const uint32_t nsync = nuq_num_sync(bucket, sync_stride);
    for (uint32_t k = 0; k < K; ++k) {
        const EncodeWorker &w = Wk.w[k];
        if (!w.bit_off || !w.words || (nsync && !w.sync))
            return NUQ_EINVAL;
        if (MODE != 1 && (!w.v || !w.norms_out || (reinterpret_cast<uintptr_t>(w.v) & 3u)))
            return NUQ_EINVAL;
        if (MODE == 1 && !w.q_in)
            return NUQ_EINVAL;
    }
    const uint64_t nb = nuq_num_buckets(d, bucket);
    const Workspace w = carve(workspace, K, nb, slot_words_for(bucket, s));
    if (w.bytes > workspace_bytes)
        return NUQ_ECAPACITY;
    uint32_t *flags = flags_ptr();
    if (!flags)
        return NUQ_EHIP;
    hipStream_t st = static_cast<hipStream_t>(stream);

    EncodeParams P{};
    P.units = w.units;
    P.staging = w.staging;
    P.flags = flags;
    const double l1 = MODE == 2 ? (double)levels[1] : std::ldexp(1.0, -(int)s);
    bool narrow = false;
    int rc = with_encode_shape<MODE>(P, K, d, bucket, s, sync_stride, l1, norm_kind == NUQ_NORM_LINF, narrow,
                                     [&](auto team_c, auto vpt_c, const TeamLdsMap &map) {
        constexpr int TEAM = decltype(team_c)::value, VPT = decltype(vpt_c)::value;
        using G = TeamGeom<TEAM>;
        const size_t lds_bytes = ((size_t)map.words * G::kTeamsPerWG + 512) * 4;            // + the code tables
        if (lds_bytes > 160 * 1024)
            return (int)NUQ_EINVAL;
        auto kern = k_encode<TEAM, VPT, MODE>;
        if (lds_bytes > 48 * 1024 &&
            hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_bytes) != hipSuccess)
            return (int)NUQ_EHIP;
        dim3 grid;
        if (!bucket_grid<TEAM>(nb, K, grid))
            return (int)NUQ_EINVAL;
        ScopedTiming timing(MODE == 1 ? NUQ_T_ENCODE : NUQ_T_QUANTIZE_ENCODE, st);
        hipLaunchKernelGGL(kern, grid, dim3(G::kWG), lds_bytes, st, P, Wk, T);
        return check_launch();
    });
    if (rc != NUQ_OK)
        return rc;

    return launch_finish(P, Wk, K, w, narrow, st);
}

bool valid_fixed(uint32_t s, uint32_t b)
{
    return b >= 3 && b <= 8 && s + 2u <= (1u << (b - 1u));
}

// MODE 0: norms + quantizer + fixed-width packing from v.  MODE 1: packing of level|sign bytes.  MODE 2: as 0 with
// the level table `levels` (host memory, s + 2 values) and the norm `norm_kind` selects.
template <int MODE>
int pack_fixed_batch(uint32_t K, const EncodeBatch &Wk, uint64_t d, uint32_t bucket, uint32_t s, uint32_t b,
                     nuq_stream_t stream, const float *levels = nullptr, uint32_t norm_kind = NUQ_NORM_L2)
{
    if (K < 1 || K > kMaxBatch || !valid_common(d, bucket, s) || !valid_fixed(s, b))
        return NUQ_EINVAL;
    LevelTable T{};
    if (MODE == 2) {
        if (!levels || !valid_levels(levels, s) || (norm_kind != NUQ_NORM_L2 && norm_kind != NUQ_NORM_LINF))
            return NUQ_EINVAL;
        for (uint32_t j = 0; j < s + 2u; ++j)
            T.lev[j] = levels[j];
    }
    for (uint32_t k = 0; k < K; ++k) {
        const EncodeWorker &w = Wk.w[k];
        if (!w.words)
            return NUQ_EINVAL;
        if (MODE != 1 && (!w.v || !w.norms_out || (reinterpret_cast<uintptr_t>(w.v) & 3u)))
            return NUQ_EINVAL;
        if (MODE == 1 && !w.q_in)
            return NUQ_EINVAL;
    }
    uint32_t *flags = flags_ptr();
    if (!flags)
        return NUQ_EHIP;
    hipStream_t st = static_cast<hipStream_t>(stream);
    EncodeParams P{};
    P.d = d;
    P.nb = nuq_num_buckets(d, bucket);
    P.bucket = bucket;
    P.s = s;
    P.flags = flags;
    P.norm_linf = norm_kind == NUQ_NORM_LINF ? 1u : 0u;
    P.stream = stream_loads(d, K);
    FixedParams F{};
    F.b = b;
    F.wpb = (bucket * b + 31u) / 32u;
    constexpr TeamUse kUse = MODE == 2 ? TeamUse::kPackTable : TeamUse::kStore;
    const bool narrow = narrow_teams<kUse>(P.nb, K, bucket, s);
    return dispatch_team<kUse>(bucket, narrow, [&](auto team_c, auto vpt_c) {
        constexpr int TEAM = decltype(team_c)::value, VPT = decltype(vpt_c)::value;
        using G = TeamGeom<TEAM>;
        P.rows = team_rows<TEAM>(bucket);
        if (b == 4 || b == 8) {             // codes go from registers to memory
            dim3 grid;
            if (!bucket_grid<TEAM>(P.nb, K, grid))
                return (int)NUQ_EINVAL;
            ScopedTiming timing(MODE == 1 ? NUQ_T_ENCODE : NUQ_T_QUANTIZE_ENCODE, st);
            if (b == 4)
                hipLaunchKernelGGL((k_pack_fixed_direct<TEAM, VPT, MODE, 4>), grid, dim3(G::kWG), 0, st, P, Wk, F, T);
            else
                hipLaunchKernelGGL((k_pack_fixed_direct<TEAM, VPT, MODE, 8>), grid, dim3(G::kWG), 0, st, P, Wk, F, T);
            return check_launch();
        }
        P.lds_words = fixed_lds_words(P.rows, TEAM, F.wpb);
        const size_t lds_bytes = (size_t)P.lds_words * 4 * G::kTeamsPerWG;
        if (lds_bytes > 160 * 1024)
            return (int)NUQ_EINVAL;
        auto kern = k_pack_fixed<TEAM, VPT, MODE>;
        if (lds_bytes > 48 * 1024 &&
            hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_bytes) != hipSuccess)
            return (int)NUQ_EHIP;
        dim3 grid;
        if (!bucket_grid<TEAM>(P.nb, K, grid))
            return (int)NUQ_EINVAL;
        ScopedTiming timing(MODE == 1 ? NUQ_T_ENCODE : NUQ_T_QUANTIZE_ENCODE, st);
        hipLaunchKernelGGL(kern, grid, dim3(G::kWG), lds_bytes, st, P, Wk, F, T);
        return check_launch();
    });
}

// Canonical code tables from code lengths (host arithmetic).  False unless the lengths describe a complete
// prefix code over the s + 2 level indices with lengths 1..15.
bool huffman_tables(const uint8_t *lengths, uint32_t s, HuffmanCode &H)
{
    H = HuffmanCode{};
    H.nsym = s + 2u;
    uint32_t next = 0, code = 0, prev_len = 0;
    bool any = false;
    for (uint32_t len = 1; len <= 15u; ++len) {
        H.offset[len] = next;
        for (uint32_t j = 0; j < H.nsym; ++j) {
            if (lengths[j] != len)
                continue;
            if (any)
                code = (code + 1u) << (len - prev_len);
            any = true;
            prev_len = len;
            if (!H.count[len])
                H.first[len] = code;
            ++H.count[len];
            H.code[j] = code;
            H.len[j] = len;
            H.sorted[next++] = j;
            H.maxlen = len;
        }
    }
    return any && next == H.nsym && code == (1u << prev_len) - 1u;
}

struct HuffmanWorkspace {
    uint32_t *units;       // bucket bit lengths
    uint64_t *chunk_sums;
    uint64_t bytes;
};

HuffmanWorkspace carve_huffman(void *base, uint64_t nb)
{
    HuffmanWorkspace w{};
    const uint64_t nb_stride = (nb + 3) & ~3ull, nchunks = (nb + kChunk - 1) / kChunk;
    uint8_t *p = static_cast<uint8_t *>(base);
    w.units = reinterpret_cast<uint32_t *>(p);
    uint64_t off = (nb_stride * 4 + 15) & ~15ull;
    w.chunk_sums = reinterpret_cast<uint64_t *>(p + off);
    off += (nchunks + 1) * 8;
    w.bytes = (off + 15) & ~15ull;
    return w;
}

// Workgroups of the persistent decode kernel that the current device holds at once (0 on error).
// `variant` indexes kDecodeKernels: 2 * (3 * table + update) + big tile.
using DecodeKernel = void (*)(DecodeParams);
constexpr DecodeKernel kDecodeKernels[] = {
    k_decode_accumulate<false, kUpdateWrite, kTileCoords>,    k_decode_accumulate<false, kUpdateWrite, kTileCoordsBig>,
    k_decode_accumulate<false, kUpdateAdd, kTileCoords>,      k_decode_accumulate<false, kUpdateAdd, kTileCoordsBig>,
    k_decode_accumulate<false, kUpdateMomentum, kTileCoords>, k_decode_accumulate<false, kUpdateMomentum, kTileCoordsBig>,
    k_decode_accumulate<true, kUpdateWrite, kTileCoords>,     k_decode_accumulate<true, kUpdateWrite, kTileCoordsBig>,
    k_decode_accumulate<true, kUpdateAdd, kTileCoords>,       k_decode_accumulate<true, kUpdateAdd, kTileCoordsBig>,
};
constexpr uint32_t kDecodeVariants = sizeof(kDecodeKernels) / sizeof(kDecodeKernels[0]);
// the same variants of the one-wave tile decoder
constexpr DecodeKernel kDecodeWaveKernels[kDecodeVariants] = {
    k_decode_wave<false, kUpdateWrite, kTileCoords>,    k_decode_wave<false, kUpdateWrite, kTileCoordsBig>,
    k_decode_wave<false, kUpdateAdd, kTileCoords>,      k_decode_wave<false, kUpdateAdd, kTileCoordsBig>,
    k_decode_wave<false, kUpdateMomentum, kTileCoords>, k_decode_wave<false, kUpdateMomentum, kTileCoordsBig>,
    k_decode_wave<true, kUpdateWrite, kTileCoords>,     k_decode_wave<true, kUpdateWrite, kTileCoordsBig>,
    k_decode_wave<true, kUpdateAdd, kTileCoords>,       k_decode_wave<true, kUpdateAdd, kTileCoordsBig>,
};

uint32_t decode_resident_workgroups(uint32_t variant, bool wave)
{
    static uint32_t cached[2][kDecodeVariants][64] = {};
    int dev = 0;
    if (variant >= kDecodeVariants || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return 0;
    uint32_t &slot = cached[wave ? 1 : 0][variant][dev];
    if (!slot) {
        int per_cu = 0, cus = 0;
        const void *kern = reinterpret_cast<const void *>(wave ? kDecodeWaveKernels[variant] : kDecodeKernels[variant]);
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, (int)(wave ? kWaveWG : kDecodeWG), 0) !=
                hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || per_cu < 1 ||
            cus < 1)
            return 0;
        slot = (uint32_t)per_cu * (uint32_t)cus;
    }
    return slot;
}

}  // namespace

extern "C" {

// Which nuq.h this library is built from (see build.py); 0: not said.
#ifndef NUQ_HEADER_KEY
#define NUQ_HEADER_KEY 0ull
#endif
extern const uint64_t nuq_header_key;
const uint64_t nuq_header_key = NUQ_HEADER_KEY;

uint64_t nuq_num_buckets(uint64_t d, uint32_t bucket)
{
    return bucket ? (d + bucket - 1) / bucket : 0;
}

uint32_t nuq_num_sync(uint32_t bucket, uint32_t sync_stride)
{
    if (!bucket || !valid_sync(sync_stride) || !sync_stride)
        return 0;
    return sync_blocks(bucket) << sync_pieces_shift(bucket, sync_stride);
}

uint32_t nuq_huffman_num_sync(uint32_t bucket, uint32_t sync_stride)
{
    return sync_stride ? (bucket + sync_stride - 1) / sync_stride - 1 : 0;
}

uint64_t nuq_max_words(uint64_t d, uint32_t bucket, uint32_t s)
{
    if (!bucket)
        return 0;
    return (d * (2u + erc_len_host(s + 1)) + 31) / 32 + nuq_num_buckets(d, bucket);
}

uint64_t nuq_encode_workspace_bytes(uint32_t K, uint64_t d, uint32_t bucket, uint32_t s)
{
    if (K < 1 || K > kMaxBatch || !valid_common(d, bucket, s))
        return 0;
    return carve(nullptr, K, nuq_num_buckets(d, bucket), slot_words_for(bucket, s)).bytes;
}

uint64_t nuq_workspace_bytes(uint64_t d, uint32_t bucket, uint32_t K)
{
    return nuq_encode_workspace_bytes(K, d, bucket, NUQ_MAX_S);
}

int nuq_bucket_norms(const float *v, uint64_t d, uint32_t bucket, float *norms, nuq_stream_t stream)
{
    if (!v || !norms || !valid_common(d, bucket, 1) || (reinterpret_cast<uintptr_t>(v) & 3u))
        return NUQ_EINVAL;
    EncodeParams P{};
    EncodeBatch Wk{};
    Wk.w[0].v = v;
    Wk.w[0].norms_out = norms;
    P.d = d;
    P.bucket = bucket;
    P.nb = nuq_num_buckets(d, bucket);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool narrow = narrow_teams<TeamUse::kStore>(P.nb, 1, bucket, 0);
    return dispatch_team<TeamUse::kStore>(bucket, narrow, [&](auto team_c, auto vpt_c) {
        constexpr int TEAM = decltype(team_c)::value, VPT = decltype(vpt_c)::value;
        dim3 grid;
        if (!bucket_grid<TEAM>(P.nb, 1, grid))
            return (int)NUQ_EINVAL;
        ScopedTiming timing(NUQ_T_NORMS, st);
        hipLaunchKernelGGL((k_bucket_norms<TEAM, VPT>), grid, dim3(TeamGeom<TEAM>::kWG), 0, st, P, Wk);
        return check_launch();
    });
}

int nuq_quantize(const float *v, uint64_t d, uint32_t bucket, uint32_t s, uint64_t seed, const float *norms,
                 uint8_t *q, nuq_stream_t stream)
{
    if (!v || !norms || !q || !valid_common(d, bucket, s) || (reinterpret_cast<uintptr_t>(v) & 3u))
        return NUQ_EINVAL;
    EncodeParams P{};
    EncodeBatch Wk{};
    Wk.w[0].v = v;
    Wk.w[0].norms_in = norms;
    Wk.w[0].q_out = q;
    Wk.w[0].seed = seed;
    P.d = d;
    P.bucket = bucket;
    P.s = s;
    P.nb = nuq_num_buckets(d, bucket);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool narrow = narrow_teams<TeamUse::kStore>(P.nb, 1, bucket, 0);
    return dispatch_team<TeamUse::kStore>(bucket, narrow, [&](auto team_c, auto vpt_c) {
        constexpr int TEAM = decltype(team_c)::value, VPT = decltype(vpt_c)::value;
        P.rows = team_rows<TEAM>(bucket);
        dim3 grid;
        if (!bucket_grid<TEAM>(P.nb, 1, grid))
            return (int)NUQ_EINVAL;
        ScopedTiming timing(NUQ_T_QUANTIZE, st);
        hipLaunchKernelGGL((k_quantize<TEAM, VPT>), grid, dim3(TeamGeom<TEAM>::kWG), 0, st, P, Wk);
        return check_launch();
    });
}

int nuq_bucket_norms_linf(const float *v, uint64_t d, uint32_t bucket, float *norms, nuq_stream_t stream)
{
    if (!v || !norms || !valid_common(d, bucket, 1) || (reinterpret_cast<uintptr_t>(v) & 3u))
        return NUQ_EINVAL;
    EncodeParams P{};
    EncodeBatch Wk{};
    Wk.w[0].v = v;
    Wk.w[0].norms_out = norms;
    P.d = d;
    P.bucket = bucket;
    P.nb = nuq_num_buckets(d, bucket);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool narrow = narrow_teams<TeamUse::kStore>(P.nb, 1, bucket, 0);
    return dispatch_team<TeamUse::kStore>(bucket, narrow, [&](auto team_c, auto vpt_c) {
        constexpr int TEAM = decltype(team_c)::value, VPT = decltype(vpt_c)::value;
        dim3 grid;
        if (!bucket_grid<TEAM>(P.nb, 1, grid))
            return (int)NUQ_EINVAL;
        ScopedTiming timing(NUQ_T_NORMS, st);
        hipLaunchKernelGGL((k_bucket_norms_linf<TEAM, VPT>), grid, dim3(TeamGeom<TEAM>::kWG), 0, st, P, Wk);
        return check_launch();
    });
}

int nuq_quantize_table(const float *v, uint64_t d, uint32_t bucket, uint32_t s, const float *levels, uint64_t seed,
                       const float *norms, uint8_t *q, nuq_stream_t stream)
{
    if (!v || !norms || !q || !levels || !valid_common(d, bucket, s) || !valid_levels(levels, s) ||
        (reinterpret_cast<uintptr_t>(v) & 3u))
        return NUQ_EINVAL;
    EncodeParams P{};
    EncodeBatch Wk{};
    LevelTable T{};
    for (uint32_t j = 0; j < s + 2u; ++j)
        T.lev[j] = levels[j];
    Wk.w[0].v = v;
    Wk.w[0].norms_in = norms;
    Wk.w[0].q_out = q;
    Wk.w[0].seed = seed;
    P.d = d;
    P.bucket = bucket;
    P.s = s;
    P.nb = nuq_num_buckets(d, bucket);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool narrow = narrow_teams<TeamUse::kStore>(P.nb, 1, bucket, 0);
    return dispatch_team<TeamUse::kStore>(bucket, narrow, [&](auto team_c, auto vpt_c) {
        constexpr int TEAM = decltype(team_c)::value, VPT = decltype(vpt_c)::value;
        P.rows = team_rows<TEAM>(bucket);
        dim3 grid;
        if (!bucket_grid<TEAM>(P.nb, 1, grid))
            return (int)NUQ_EINVAL;
        ScopedTiming timing(NUQ_T_QUANTIZE, st);
        hipLaunchKernelGGL((k_quantize_table<TEAM, VPT>), grid, dim3(TeamGeom<TEAM>::kWG), 0, st, P, Wk, T);
        return check_launch();
    });
}

int nuq_encode(const uint8_t *q, uint64_t d, uint32_t bucket, uint32_t s, uint32_t sync_stride, uint64_t *bit_off,
               uint32_t *words, uint64_t words_cap, uint32_t *sync, void *workspace, uint64_t workspace_bytes,
               nuq_stream_t stream)
{
    EncodeBatch Wk{};
    Wk.w[0].q_in = q;
    Wk.w[0].bit_off = bit_off;
    Wk.w[0].words = words;
    Wk.w[0].words_cap = words_cap;
    Wk.w[0].sync = sync;
    return encode_batch<1>(1, Wk, d, bucket, s, sync_stride, workspace, workspace_bytes, stream);
}

int nuq_quantize_encode(const float *v, uint64_t d, uint32_t bucket, uint32_t s, uint64_t seed,
                        uint32_t sync_stride, float *norms, uint64_t *bit_off, uint32_t *words, uint64_t words_cap,
                        uint32_t *sync, void *workspace, uint64_t workspace_bytes, nuq_stream_t stream)
{
    EncodeBatch Wk{};
    Wk.w[0].v = v;
    Wk.w[0].seed = seed;
    Wk.w[0].norms_out = norms;
    Wk.w[0].bit_off = bit_off;
    Wk.w[0].words = words;
    Wk.w[0].words_cap = words_cap;
    Wk.w[0].sync = sync;
    return encode_batch<0>(1, Wk, d, bucket, s, sync_stride, workspace, workspace_bytes, stream);
}

int nuq_quantize_encode_static(const float *v, uint64_t d, uint32_t bucket, uint32_t s, uint64_t seed,
                               uint32_t sync_stride, float *norms, uint64_t *bit_off, uint32_t *words,
                               uint64_t words_cap, uint32_t *sync, nuq_stream_t stream)
{
    const uint64_t need = nuq_encode_workspace_bytes(1, d, bucket, s);
    if (!need)
        return NUQ_EINVAL;
    if (need > NUQ_STATIC_WORKSPACE_BYTES)
        return NUQ_ECAPACITY;
    void *ws = static_workspace_ptr();
    if (!ws)
        return NUQ_EHIP;
    return nuq_quantize_encode(v, d, bucket, s, seed, sync_stride, norms, bit_off, words, words_cap, sync, ws,
                               NUQ_STATIC_WORKSPACE_BYTES, stream);
}

int nuq_quantize_encode_batch(uint32_t K, const float *const *v, const uint64_t *seeds, uint64_t d, uint32_t bucket,
                              uint32_t s, uint32_t sync_stride, float *const *norms, uint64_t *const *bit_off,
                              uint32_t *const *words, const uint64_t *words_cap, uint32_t *const *sync,
                              void *workspace, uint64_t workspace_bytes, nuq_stream_t stream)
{
    if (K < 1 || K > kMaxBatch || !v || !seeds || !norms || !bit_off || !words || !words_cap)
        return NUQ_EINVAL;
    EncodeBatch Wk{};
    for (uint32_t k = 0; k < K; ++k) {
        Wk.w[k].v = v[k];
        Wk.w[k].seed = seeds[k];
        Wk.w[k].norms_out = norms[k];
        Wk.w[k].bit_off = bit_off[k];
        Wk.w[k].words = words[k];
        Wk.w[k].words_cap = words_cap[k];
        Wk.w[k].sync = sync ? sync[k] : nullptr;
    }
    return encode_batch<0>(K, Wk, d, bucket, s, sync_stride, workspace, workspace_bytes, stream);
}

// Coordinates of a tile of the decoders that have an index (update: what the output stage does with the sums, a kUpdate).
//
// Tiles of 4096 coordinates (32 KB of fp64, four workgroups per CU instead of eight) where the usual 2048 would
// give the 64 parsing lanes at most 32 units: parts of large buckets of few workers whose pieces are long, or may be (level
// tables).  The parse of long pieces is bound by instruction issue, so one full wave per SIMD gets through more records
// than two half-empty ones (four messages in buckets of 8192 at s = 7, stride 512, 3 M coordinates 52.0 us, in tiles of 2048
// 56.4; of 16384 at 256, 205 records to a piece, 27.2 and 30.1).  Up to about 128 records to a piece (with the main scheme
// 0.8 x 2^s / sqrt(bucket) of the coordinates are nonzero on average, and never more than all) more waves and half the result for
// each count for more: at s = 3, stride 256, 65 537 coordinates 7.98 -> 7.04 us with tiles of 2048, 6 M 13.9 -> 12.6, 60 M 69.1 ->
// 65.6; two messages in buckets of 20000 at s = 7, stride 128, 3 M 16.9 -> 15.6, of 4096, 1 M 16.3 -> 14.7; 8192 at s = 5, stride 256,
// 0.3 M 17.2 -> 15.7; momentum on one of 5000 at s = 8, 6 M 86.9 -> 72.2.  (Two dense messages at s = 14, stride 128, 1 M or less are
// 10 % slower so: 18.3 and 20.7.)  With a full chip the line lies lower (58.4 and 59.2 us on 20 M of 8192 at s = 5, 72 records).
// Small buckets: only where they fill the tile, 2048 coordinates have at most 16 units (4 x 16.8 M coordinates in buckets
// of 512 at stride 512 84 -> 78 us, two messages at 256 48 -> 44; with 32 units 50 -> 52), there is a tile for every CU
// (0.3 M coordinates, exponential levels at s = 7, both directions 65.8 -> 69.5 with tiles of 4096) and the result is
// written: what the other updates read takes registers for twice the coordinates, which leaves a wave per SIMD (17 M
// coordinates of two messages in buckets of 512, momentum 52 -> 67 us; 10 M of one in buckets of 1024 28 -> 34).
static uint32_t decode_tile_coords(uint32_t K, uint64_t d, uint32_t bucket, uint32_t s, uint32_t sync_stride, bool table,
                                   uint32_t update)
{
    if (!nuq_num_sync(bucket, sync_stride))
        return kTileCoords;
    const uint32_t pieces = 1u << sync_pieces_shift(bucket, sync_stride);       // per block of the index and message
    if (bucket >= kTileCoordsBig) {
        const double records = sync_stride * std::min(1.0, 0.8 * std::ldexp(1.0, (int)s) / std::sqrt((double)bucket));
        const bool short_pieces = !table && records <= (d < (1ull << 24) ? 128.0 : 64.0);
        return !short_pieces && K * pieces <= 32u ? kTileCoordsBig : kTileCoords;
    }
    return kTileCoordsBig % bucket == 0 && kTileCoordsBig / bucket * K <= kMaxStreams && update == kUpdateWrite &&
                   d >= 256ull * kTileCoordsBig && kTileCoords / bucket * K * pieces <= 16u
               ? kTileCoordsBig
               : kTileCoords;
}

// levels: nullptr for the levels 2^(j-1-s), else the s + 2 values of a level table (host memory).
static int decode_accumulate_any(uint32_t K, const float *const *norms, const uint64_t *const *bit_off,
                                 const uint32_t *const *words, const uint64_t *words_len,
                                 const uint32_t *const *sync, uint64_t d,
                                 uint32_t bucket, uint32_t s, uint32_t sync_stride, const float *levels, float scale,
                                 int accumulate, float *out, nuq_stream_t stream,
                                 const MomentumParams *momentum = nullptr)
{
    if (K < 1 || K > NUQ_MAX_WORKERS || !norms || !bit_off || !words || !words_len || !out ||
        !valid_common(d, bucket, s) ||
        !valid_sync(sync_stride) || (levels && !valid_levels(levels, s)))
        return NUQ_EINVAL;
    const uint32_t nsync = nuq_num_sync(bucket, sync_stride);
    if (nsync && !sync)
        return NUQ_EINVAL;
    DecodeParams P{};
    for (uint32_t k = 0; k < K; ++k) {
        if (!norms[k] || !bit_off[k] || !words[k] || (nsync && !sync[k]))
            return NUQ_EINVAL;
        P.norms[k] = norms[k];
        P.bit_off[k] = bit_off[k];
        P.words[k] = words[k];
        P.words_bits[k] = words_len[k] > (UINT64_MAX >> 5) ? UINT64_MAX : words_len[k] << 5;
        P.sync[k] = nsync ? sync[k] : nullptr;
    }
    uint32_t *flags = flags_ptr();
    if (!flags)
        return NUQ_EHIP;
    P.out = out;
    P.flags = flags;
    P.d = d;
    P.nb = nuq_num_buckets(d, bucket);
    P.K = K;
    P.bucket = bucket;
    P.s = s;
    P.nsync = nsync;
    P.nseg = nsync ? nsync : 1;                 // units (pieces) per bucket and worker
    P.pieces_shift = nsync ? sync_pieces_shift(bucket, sync_stride) : 0;
    P.scale = scale;
    if (momentum && levels)
        return NUQ_EINVAL;
    if (K == 1 && !levels && !momentum && (nsync || bucket <= 512)) {
        // k_decode_one costs the parse and the result; k_decode_single clears the result and scatters the values, which costs
        // little where they are few and the result stays in the 256 MB last-level cache in between.  With fewer than a coordinate
        // in seven nonzero (0.8 x 2^s / sqrt(bucket) of them are, on average) it is faster from 2 M to 64 M coordinates: 27 M in
        // buckets of 8192 at s = 3 17 %, 41 M of 10 000 at s = 1 38 %; below that launches weigh more, beyond it memory does (124 M of
        // 1000 at s = 3 takes 1.6 times as long).  So it is where an index piece has much less than a stride's coordinates (a
        // bucket just above a block or a power of two of strides: 44 M of 513 at stride 128 53 us and 93), and at stride 64, where
        // a wave's 64 pieces are a fourth of what its bytes hold, below 4 M (5 % in the mean).
        const uint32_t filled = nsync ? std::min(sync_stride, bucket) : 0u;
        const bool one = d >= (1ull << 26) || (10ull * bucket >= 6ull * P.nseg * filled && (sync_stride > 64u || d >= (1ull << 22)) &&
                                               (d < (1ull << 21) || bucket <= (32ull << (2u * s))));
        if (!accumulate && nsync && bucket >= kOneMinBucket && one) {
            // One message, written: up to 64 pieces per wave, as many blocks of 2048 coordinates (whole buckets below that)
            // as 16 KB of bytes hold, less three that the first float4 group may begin before the first of them; no more than one
            // and another for every 1024 blocks that there are, which leaves 512 waves or more to a message of that many (1 M
            // coordinates: 14.3 us with eight blocks each, 8.0 with one).  One for every whole 1024, hence 1024 waves, is slower
            // where pieces are long: 1 M at s = 7 in buckets of 512 49.0 and 72.5 us, 3.8 M at s = 5 in 4096 16.8 and 30.3.
            constexpr uint64_t kOneWaves = 1024;
            const uint32_t span = std::min(bucket, 1u << kSyncBlockShift);
            const uint64_t nblocks = P.nb * (P.nseg >> P.pieces_shift);
            P.segs_per_tile = (uint32_t)std::min<uint64_t>(
                std::min(64u >> P.pieces_shift, (kOneCoords - (bucket % 4u ? 3u : 0u)) / span), (nblocks + kOneWaves) / kOneWaves);
            const uint64_t wgs = (nblocks + P.segs_per_tile - 1) / P.segs_per_tile;
            if (wgs > 0x7fffffffull)
                return NUQ_EINVAL;
            ScopedTiming timing(NUQ_T_DECODE, static_cast<hipStream_t>(stream));
            hipLaunchKernelGGL(k_decode_one, dim3((uint32_t)wgs), dim3(kWave), 0, static_cast<hipStream_t>(stream), P);
            return check_launch();
        }
        // one message: a lane per (bucket, sync segment), values stored directly (k_decode_single)
        const uint64_t wgs = (P.nb * P.nseg + kSingleWG - 1) / kSingleWG;
        if (wgs > 0x7fffffffull)
            return NUQ_EINVAL;
        ScopedTiming timing(NUQ_T_DECODE, static_cast<hipStream_t>(stream));
        if (accumulate)
            hipLaunchKernelGGL(k_decode_single<kUpdateAdd>, dim3((uint32_t)wgs), dim3(kSingleWG), 0,
                               static_cast<hipStream_t>(stream), P);
        else
            hipLaunchKernelGGL(k_decode_single<kUpdateWrite>, dim3((uint32_t)wgs), dim3(kSingleWG), 0,
                               static_cast<hipStream_t>(stream), P);
        return check_launch();
    }
    const uint32_t update = momentum ? (uint32_t)kUpdateMomentum : accumulate ? (uint32_t)kUpdateAdd : (uint32_t)kUpdateWrite;
    const uint32_t tile_coords = decode_tile_coords(K, d, bucket, s, sync_stride, levels != nullptr, update);
    const uint32_t variant = 2u * ((levels ? 3u : 0u) + update) + (tile_coords == kTileCoordsBig ? 1u : 0u);
    if (momentum) {
        P.yl = momentum->yl;
        P.alpha = momentum->alpha;
        P.la = momentum->l * momentum->alpha;
        P.mu = momentum->mu;
    }
    uint64_t ntiles;
    uint32_t max_streams;
    if (bucket <= kTileCoords) {
        const uint32_t by_size = tile_coords / bucket, by_streams = kMaxStreams / K;
        P.buckets_per_tile = by_size < by_streams ? by_size : by_streams;
        P.tiles_per_bucket = 1;
        P.tile_coords = P.buckets_per_tile * bucket;
        P.segs_per_tile = P.nseg;
        ntiles = (P.nb + P.buckets_per_tile - 1) / P.buckets_per_tile;
        max_streams = P.buckets_per_tile * K;
    } else {
        P.buckets_per_tile = 0;
        P.tile_coords = tile_coords;
        P.tiles_per_bucket = (bucket + tile_coords - 1) / tile_coords;
        P.segs_per_tile = nsync ? (tile_coords >> kSyncBlockShift) << P.pieces_shift : 1;
        ntiles = P.nb * P.tiles_per_bucket;
        max_streams = K;
    }
    if (ntiles > 0x7fffffffull)
        return NUQ_EINVAL;
    P.ntiles = (uint32_t)ntiles;
    P.xcd_base = P.ntiles / 8u;
    P.xcd_rem = P.ntiles % 8u;
    // lanes (of the preparing wave) per stream for the copy of its words: the largest power of two that gives
    // every stream a group
    P.lanes_shift = 0;
    while ((2u << P.lanes_shift) * max_streams <= 64u)
        ++P.lanes_shift;
    P.stream_cap = kWordsPerLane << P.lanes_shift;
    // An odd stride when a tile has many streams (small buckets): lanes of different streams stand at like offsets,
    // and with a stride of 8 or 16 words they would read the same few banks (config 5: -5 %).  With few, long
    // streams the word given up costs more than the conflicts (config 4: +4 %), so those keep the full stride.
    P.stream_stride = max_streams >= 16u ? P.stream_cap - 1u : P.stream_cap;
    // One wave per workgroup where a tile holds at most 64 pieces and each stream's pieces fit the lanes that copy it
    // (every usual geometry with an index); the two-wave kernel takes the rest (no index, many workers, fine strides).
    const bool wave = nsync && max_streams <= 64u && P.segs_per_tile <= (1u << P.lanes_shift);
    if (wave)
        P.parts_shift = P.lanes_shift - log2u(P.segs_per_tile);
    uint32_t resident = decode_resident_workgroups(variant, wave);
    if (!resident)
        return NUQ_EHIP;
    resident &= ~7u;                            // a multiple of the eight XCDs (see xcd_tile)
    if (!resident)
        resident = 8u;
    // Every resident workgroup slot is used.  Workgroups walk tiles with stride `grid`, so the first
    // ntiles mod grid of them get one tile more than the rest: those are the workgroups that arrive first on their
    // CUs, whose parsing waves are the oldest on their SIMDs and run faster than the later ones.
    const uint32_t grid = P.ntiles < resident ? P.ntiles : resident;
    // Pieces of more words than a row of decode_wave, one lane each: row after row, the wave waits at the end of each for the
    // lane with most records, and pays a round trip; from global memory it does not, as long as the pieces of the waves on a CU
    // (256 of them) stay in its cache of 32 KB, of which 24 are counted on.  With 64 words and more to a piece a line per lane
    // is what counts, hence no bound on the piece then.  Rows and global memory in turn, written: 4 x 2.7 M coordinates in buckets
    // of 8192 at s = 5, stride 256 (13 words) 16.3 and 15.0 us, 4 x 7.6 M at s = 6 (19) 39.1 and 37.3, 5 x 0.2 M at s = 10, stride
    // 512 (103 words, a wave per CU) 58.1 and 54.9; beyond the bound 4 x 14.7 M in buckets of 4096 at s = 7 (30) 103 and 111, 8 x
    // 12.3 M at s = 10 (105) 177 and 301.  Where several lanes load a piece's longer row, and in small buckets, rows are faster
    // throughout (4 x 0.4 M at s = 7, stride 512 51.4 and 53.3; 7 x 0.8 M in buckets of 256 16.9 and 18.0).
    if (wave && !P.parts_shift && bucket > 512u) {
        constexpr uint32_t kDirectWords = 24u * 1024u / 4u;
        P.direct_words = kDirectWords / (max_streams * P.segs_per_tile * ((grid + 255u) / 256u));
        if (P.direct_words >= 64u)
            P.direct_words = ~0u;
    }
    ScopedTiming timing(NUQ_T_DECODE, static_cast<hipStream_t>(stream));
    if (levels)
        for (uint32_t j = 0; j < s + 2u; ++j)
            P.lev[j] = levels[j];
    if (wave)
        hipLaunchKernelGGL(kDecodeWaveKernels[variant], dim3(grid), dim3(kWaveWG), 0, static_cast<hipStream_t>(stream), P);
    else
        hipLaunchKernelGGL(kDecodeKernels[variant], dim3(grid), dim3(kDecodeWG), 0, static_cast<hipStream_t>(stream), P);
    return check_launch();
}

int nuq_quantize_encode_table_batch(uint32_t K, const float *const *v, const uint64_t *seeds, uint64_t d,
                                    uint32_t bucket, uint32_t s, const float *levels, uint32_t norm_kind,
                                    uint32_t sync_stride, float *const *norms, uint64_t *const *bit_off,
                                    uint32_t *const *words, const uint64_t *words_cap, uint32_t *const *sync,
                                    void *workspace, uint64_t workspace_bytes, nuq_stream_t stream)
{
    if (K < 1 || K > kMaxBatch || !v || !seeds || !norms || !bit_off || !words || !words_cap || !levels)
        return NUQ_EINVAL;
    EncodeBatch Wk{};
    for (uint32_t k = 0; k < K; ++k) {
        Wk.w[k].v = v[k];
        Wk.w[k].seed = seeds[k];
        Wk.w[k].norms_out = norms[k];
        Wk.w[k].bit_off = bit_off[k];
        Wk.w[k].words = words[k];
        Wk.w[k].words_cap = words_cap[k];
        Wk.w[k].sync = sync ? sync[k] : nullptr;
    }
    return encode_batch<2>(K, Wk, d, bucket, s, sync_stride, workspace, workspace_bytes, stream, levels, norm_kind);
}

int nuq_decode_accumulate(uint32_t K, const float *const *norms, const uint64_t *const *bit_off,
                          const uint32_t *const *words, const uint64_t *words_len, const uint32_t *const *sync,
                          uint64_t d, uint32_t bucket, uint32_t s, uint32_t sync_stride, float scale, int accumulate,
                          float *out, nuq_stream_t stream)
{
    return decode_accumulate_any(K, norms, bit_off, words, words_len, sync, d, bucket, s, sync_stride, nullptr, scale,
                                 accumulate, out, stream);
}

int nuq_decode_accumulate_table(uint32_t K, const float *const *norms, const uint64_t *const *bit_off,
                                const uint32_t *const *words, const uint64_t *words_len,
                                const uint32_t *const *sync, uint64_t d, uint32_t bucket, uint32_t s,
                                uint32_t sync_stride, const float *levels, float scale, int accumulate, float *out,
                                nuq_stream_t stream)
{
    if (!levels)
        return NUQ_EINVAL;
    return decode_accumulate_any(K, norms, bit_off, words, words_len, sync, d, bucket, s, sync_stride, levels, scale,
                                 accumulate, out, stream);
}

uint64_t nuq_fixed_words(uint64_t d, uint32_t bucket, uint32_t b)
{
    if (!bucket || b < 3 || b > 8)
        return 0;
    return nuq_num_buckets(d, bucket) * (((uint64_t)bucket * b + 31) / 32);
}

int nuq_pack_fixed(const uint8_t *q, uint64_t d, uint32_t bucket, uint32_t s, uint32_t b, uint32_t *packed,
                   nuq_stream_t stream)
{
    EncodeBatch Wk{};
    Wk.w[0].q_in = q;
    Wk.w[0].words = packed;
    return pack_fixed_batch<1>(1, Wk, d, bucket, s, b, stream);
}

int nuq_quantize_pack_fixed_batch(uint32_t K, const float *const *v, const uint64_t *seeds, uint64_t d,
                                  uint32_t bucket, uint32_t s, uint32_t b, float *const *norms,
                                  uint32_t *const *packed, nuq_stream_t stream)
{
    if (K < 1 || K > kMaxBatch || !v || !seeds || !norms || !packed)
        return NUQ_EINVAL;
    EncodeBatch Wk{};
    for (uint32_t k = 0; k < K; ++k) {
        Wk.w[k].v = v[k];
        Wk.w[k].seed = seeds[k];
        Wk.w[k].norms_out = norms[k];
        Wk.w[k].words = packed[k];
    }
    return pack_fixed_batch<0>(K, Wk, d, bucket, s, b, stream);
}

int nuq_quantize_pack_fixed_table_batch(uint32_t K, const float *const *v, const uint64_t *seeds, uint64_t d,
                                        uint32_t bucket, uint32_t s, const float *levels, uint32_t norm_kind, uint32_t b,
                                        float *const *norms, uint32_t *const *packed, nuq_stream_t stream)
{
    if (K < 1 || K > kMaxBatch || !v || !seeds || !norms || !packed || !levels)
        return NUQ_EINVAL;
    EncodeBatch Wk{};
    for (uint32_t k = 0; k < K; ++k) {
        Wk.w[k].v = v[k];
        Wk.w[k].seed = seeds[k];
        Wk.w[k].norms_out = norms[k];
        Wk.w[k].words = packed[k];
    }
    return pack_fixed_batch<2>(K, Wk, d, bucket, s, b, stream, levels, norm_kind);
}

static int unpack_accumulate_fixed_any(uint32_t K, const float *const *norms, const uint32_t *const *packed, uint64_t d,
                                       uint32_t bucket, uint32_t s, const float *levels, uint32_t b, float scale,
                                       int accumulate, float *out, nuq_stream_t stream)
{
    if (K < 1 || K > NUQ_MAX_WORKERS || !norms || !packed || !out || !valid_common(d, bucket, s) ||
        !valid_fixed(s, b) || (levels && !valid_levels(levels, s)))
        return NUQ_EINVAL;
    UnpackParams P{};
    if (levels) {
        P.use_levels = 1u;
        for (uint32_t j = 0; j < s + 2u; ++j)
            P.lev[j] = levels[j];
    }
    for (uint32_t k = 0; k < K; ++k) {
        if (!norms[k] || !packed[k])
            return NUQ_EINVAL;
        P.norms[k] = norms[k];
        P.packed[k] = packed[k];
    }
    uint32_t *flags = flags_ptr();
    if (!flags)
        return NUQ_EHIP;
    P.out = out;
    P.flags = flags;
    P.d = d;
    P.K = K;
    P.bucket = bucket;
    P.s = s;
    P.b = b;
    P.wpb = (bucket * b + 31u) / 32u;
    P.scale = scale;
    P.accumulate = accumulate;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool aligned_out = (reinterpret_cast<uintptr_t>(out) & 15u) == 0;
    if ((b == 4u || b == 8u) && bucket % (32u / b) == 0 && aligned_out) {
        // whole words per bucket, and the value tables of the buckets a workgroup can touch fit in 16 KB
        const uint32_t span = unpack_direct_coords(b);
        const uint64_t nb = nuq_num_buckets(d, bucket);
        const bool tiled = span % bucket == 0 || bucket % span == 0;
        const uint64_t tabs = std::min<uint64_t>(nb, tiled ? std::max(1u, span / bucket) : span / bucket + 2u);
        const uint64_t lut_bytes = tabs * K * fixed_lut_entries(b) * sizeof(double);
        const uint64_t blocks = (d + span - 1) / span;
        if (lut_bytes <= 16384u) {
            if (blocks > 0x7fffffffull)
                return NUQ_EINVAL;
            P.lut_tabs = (uint32_t)tabs;
            const bool one = bucket % (b == 4u ? 512u : 256u) == 0;
            auto kern = b == 4u ? (one ? k_unpack_accumulate_fixed_direct<4, true> : k_unpack_accumulate_fixed_direct<4, false>)
                                : (one ? k_unpack_accumulate_fixed_direct<8, true> : k_unpack_accumulate_fixed_direct<8, false>);
            if (b == 8u && K <= 2u)
                kern = one ? k_unpack_accumulate_fixed_direct<8, true, true> : k_unpack_accumulate_fixed_direct<8, false, true>;
            ScopedTiming timing(NUQ_T_DECODE, st);
            hipLaunchKernelGGL(kern, dim3((uint32_t)blocks), dim3(256), (uint32_t)lut_bytes, st, P);
            return check_launch();
        }
    }
    const bool wide = bucket % 32u == 0 && aligned_out;
    const uint64_t threads = wide ? (d + 31) / 32 : d;
    const uint64_t blocks = (threads + 255) / 256;
    if (blocks > 0x7fffffffull)
        return NUQ_EINVAL;
    ScopedTiming timing(NUQ_T_DECODE, st);
    const dim3 grid((uint32_t)blocks);
    if (!wide) {
        hipLaunchKernelGGL(k_unpack_accumulate_fixed1, grid, dim3(256), 0, st, P);
    } else {
        // Tables of code values in LDS when those of the buckets a workgroup (8192 coordinates) can touch fit in
        // 16 KB beside the 33 KB output tile (three workgroups per CU at worst); else the arithmetic variant.
        const uint64_t nb = nuq_num_buckets(d, bucket);
        const bool tiled = 8192u % bucket == 0 || bucket % 8192u == 0;
        const uint64_t tabs = std::min<uint64_t>(nb, tiled ? std::max(1u, 8192u / bucket) : 8192u / bucket + 2u);
        const uint64_t lut_bytes = tabs * K * fixed_lut_entries(b) * sizeof(double);
        const bool lut = lut_bytes <= 16384u;
        P.lut_tabs = (uint32_t)tabs;
        const uint32_t dyn = lut ? (uint32_t)lut_bytes : 0u;
#define NUQ_LAUNCH_UNPACK(B)                                                                                   \
    do {                                                                                                       \
        if (lut)                                                                                               \
            hipLaunchKernelGGL((k_unpack_accumulate_fixed32<B, true>), grid, dim3(256), dyn, st, P);           \
        else                                                                                                   \
            hipLaunchKernelGGL((k_unpack_accumulate_fixed32<B, false>), grid, dim3(256), 0, st, P);            \
    } while (0)
        switch (b) {
        case 3: NUQ_LAUNCH_UNPACK(3); break;
        case 5: NUQ_LAUNCH_UNPACK(5); break;
        case 6: NUQ_LAUNCH_UNPACK(6); break;
        case 7: NUQ_LAUNCH_UNPACK(7); break;
        // the tables of 4- and 8-bit codes did not fit above, and this kernel's workgroups touch no fewer buckets
        case 4: hipLaunchKernelGGL((k_unpack_accumulate_fixed32<4, false>), grid, dim3(256), 0, st, P); break;
        default: hipLaunchKernelGGL((k_unpack_accumulate_fixed32<8, false>), grid, dim3(256), 0, st, P); break;
        }
#undef NUQ_LAUNCH_UNPACK
    }
    return check_launch();
}

int nuq_unpack_accumulate_fixed(uint32_t K, const float *const *norms, const uint32_t *const *packed, uint64_t d,
                                uint32_t bucket, uint32_t s, uint32_t b, float scale, int accumulate, float *out,
                                nuq_stream_t stream)
{
    return unpack_accumulate_fixed_any(K, norms, packed, d, bucket, s, nullptr, b, scale, accumulate, out, stream);
}

int nuq_unpack_accumulate_fixed_table(uint32_t K, const float *const *norms, const uint32_t *const *packed, uint64_t d,
                                      uint32_t bucket, uint32_t s, const float *levels, uint32_t b, float scale,
                                      int accumulate, float *out, nuq_stream_t stream)
{
    if (!levels)
        return NUQ_EINVAL;
    return unpack_accumulate_fixed_any(K, norms, packed, d, bucket, s, levels, b, scale, accumulate, out, stream);
}


int nuq_level_histogram(const uint8_t *q, uint64_t d, uint64_t *hist, nuq_stream_t stream)
{
    if (!q || !hist || d < 1)
        return NUQ_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, st, reinterpret_cast<unsigned long long *>(hist), 16u);
    const uint64_t blocks = (d + 256ull * 64 - 1) / (256ull * 64);
    hipLaunchKernelGGL(k_level_histogram, dim3((uint32_t)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, st, q, d,
                       reinterpret_cast<unsigned long long *>(hist));
    return check_launch();
}

int nuq_huffman_lengths(const uint64_t *hist, uint32_t s, uint8_t *lengths)
{
    if (!hist || !lengths || s < 1 || s > NUQ_MAX_S)
        return NUQ_EINVAL;
    // Huffman's algorithm on the weights hist[j] + 1 (Sec. 5, "Efficient Encoding"), as a merge of two queues: the
    // leaves sorted by (weight, symbol), and the merged nodes in order of creation, whose weights never decrease.
    // The next smallest node is at the front of one of the queues; of two equal weights the leaf goes first, which
    // is the order (weight, id) with leaves numbered before merged nodes.
    const uint32_t nsym = s + 2u;
    uint32_t leaf[16];                  // symbols, sorted
    for (uint32_t j = 0; j < nsym; ++j)
        leaf[j] = j;
    std::stable_sort(leaf, leaf + nsym, [&](uint32_t x, uint32_t y) { return hist[x] < hist[y]; });
    uint64_t merged_weight[16];
    uint32_t kid[16][2];                // children of merged node m: a symbol, or 16 + a merged node
    uint32_t nl = 0, nm_front = 0, nm = 0;
    auto take = [&](uint64_t &weight) {
        const bool from_leaves =
            nl < nsym && (nm_front == nm || hist[leaf[nl]] + 1u <= merged_weight[nm_front]);
        if (from_leaves) {
            weight = hist[leaf[nl]] + 1u;
            return leaf[nl++];
        }
        weight = merged_weight[nm_front];
        return 16u + nm_front++;
    };
    for (uint32_t m = 0; m + 1u < nsym; ++m) {
        uint64_t w0, w1;
        kid[m][0] = take(w0);
        kid[m][1] = take(w1);
        merged_weight[m] = w0 + w1;
        nm = m + 1u;
    }
    // depths from the root (the last merged node) down
    uint32_t depth[16] = {0};
    for (uint32_t m = nsym - 1u; m-- > 0u;)
        for (uint32_t c = 0; c < 2u; ++c) {
            if (kid[m][c] >= 16u)
                depth[kid[m][c] - 16u] = depth[m] + 1u;
            else
                lengths[kid[m][c]] = (uint8_t)(depth[m] + 1u);
        }
    return NUQ_OK;
}

uint64_t nuq_huffman_max_words(uint64_t d, uint32_t bucket)
{
    if (!bucket)
        return 0;
    return (d * 16 + 31) / 32 + nuq_num_buckets(d, bucket);
}

uint64_t nuq_encode_huffman_workspace_bytes(uint64_t d, uint32_t bucket)
{
    if (!bucket)
        return 0;
    return carve_huffman(nullptr, nuq_num_buckets(d, bucket)).bytes;
}

int nuq_encode_huffman(const uint8_t *q, uint64_t d, uint32_t bucket, uint32_t s, uint32_t sync_stride,
                       const uint8_t *lengths, uint64_t *bit_off, uint32_t *words, uint64_t words_cap,
                       uint32_t *sync, void *workspace, uint64_t workspace_bytes, nuq_stream_t stream)
{
    if (!q || !lengths || !bit_off || !words || !workspace || !valid_common(d, bucket, s) ||
        !valid_sync(sync_stride) || (reinterpret_cast<uintptr_t>(workspace) & 15u))
        return NUQ_EINVAL;
    const uint32_t nsync = nuq_huffman_num_sync(bucket, sync_stride);
    if (nsync && !sync)
        return NUQ_EINVAL;
    HuffmanCode H;
    if (!huffman_tables(lengths, s, H))
        return NUQ_EINVAL;
    const uint64_t nb = nuq_num_buckets(d, bucket);
    const HuffmanWorkspace w = carve_huffman(workspace, nb);
    if (w.bytes > workspace_bytes)
        return NUQ_ECAPACITY;
    uint32_t *flags = flags_ptr();
    if (!flags)
        return NUQ_EHIP;
    hipStream_t st = static_cast<hipStream_t>(stream);
    EncodeParams P{};
    EncodeBatch Wk{};
    Wk.w[0].q_in = q;
    Wk.w[0].bit_off = bit_off;
    Wk.w[0].words = words;
    Wk.w[0].words_cap = words_cap;
    Wk.w[0].sync = sync;
    P.d = d;
    P.nb = nb;
    P.nb_stride = (nb + 3) & ~3ull;
    P.bucket = bucket;
    P.s = s;
    P.sync_shift = nsync ? log2u(sync_stride) : 0;
    P.nsync = nsync;
    P.units = w.units;
    P.flags = flags;
    const uint64_t nchunks = (nb + kChunk - 1) / kChunk;
    const bool narrow = narrow_teams<TeamUse::kStore>(P.nb, 1, bucket, 0);
    return dispatch_team<TeamUse::kStore>(bucket, narrow, [&](auto team_c, auto vpt_c) {
        constexpr int TEAM = decltype(team_c)::value, VPT = decltype(vpt_c)::value;
        using G = TeamGeom<TEAM>;
        P.rows = team_rows<TEAM>(bucket);
        P.lds_words = huffman_lds_words(P.rows, TEAM, bucket, nsync);
        const size_t lds_bytes = (size_t)P.lds_words * 4 * G::kTeamsPerWG;
        if (lds_bytes > 160 * 1024)
            return (int)NUQ_EINVAL;
        auto emit = k_huffman_emit<TEAM, VPT>;
        if (lds_bytes > 48 * 1024 &&
            hipFuncSetAttribute(reinterpret_cast<const void *>(emit), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_bytes) != hipSuccess)
            return (int)NUQ_EHIP;
        dim3 grid;
        if (!bucket_grid<TEAM>(nb, 1, grid))
            return (int)NUQ_EINVAL;
        hipLaunchKernelGGL((k_huffman_lens<TEAM, VPT>), grid, dim3(G::kWG), 0, st, P, Wk, H);
        hipLaunchKernelGGL(k_chunk_sums<true>, dim3((uint32_t)nchunks, 1), dim3(256), 0, st, w.units, nb, P.nb_stride, nchunks,
                           w.chunk_sums);
        hipLaunchKernelGGL(k_chunk_scan, dim3(1), dim3(256), 0, st, w.chunk_sums, nchunks);
        hipLaunchKernelGGL(k_bit_offsets, dim3((uint32_t)nchunks), dim3(256), 0, st, w.units, nb, w.chunk_sums, bit_off);
        ScopedTiming timing(NUQ_T_ENCODE, st);
        hipLaunchKernelGGL(emit, grid, dim3(G::kWG), lds_bytes, st, P, Wk, H);
        return check_launch();
    });
}

// Staging words per bucket for the fused Huffman encoder: every coordinate at the longest codeword (s + 1 bits) and a
// sign bit.
uint32_t huffman_slot_words(uint32_t bucket, uint32_t s)
{
    const uint64_t bits = (uint64_t)bucket * (s + 2u);
    return (uint32_t)(((bits + 31) / 32 + 3) & ~3ull);
}

uint64_t nuq_encode_huffman_batch_workspace_bytes(uint32_t K, uint64_t d, uint32_t bucket, uint32_t s)
{
    if (K < 1 || K > kMaxBatch || !valid_common(d, bucket, s))
        return 0;
    return carve(nullptr, K, nuq_num_buckets(d, bucket), huffman_slot_words(bucket, s)).bytes;
}

int nuq_quantize_encode_huffman_batch(uint32_t K, const float *const *v, const uint64_t *seeds, uint64_t d,
                                      uint32_t bucket, uint32_t s, uint32_t sync_stride, const uint8_t *lengths,
                                      float *const *norms, uint64_t *const *bit_off, uint32_t *const *words,
                                      const uint64_t *words_cap, uint32_t *const *sync, void *workspace,
                                      uint64_t workspace_bytes, nuq_stream_t stream)
{
    if (K < 1 || K > kMaxBatch || !v || !seeds || !norms || !bit_off || !words || !words_cap || !lengths ||
        !workspace || (reinterpret_cast<uintptr_t>(workspace) & 15u) || !valid_common(d, bucket, s) ||
        !valid_sync(sync_stride))
        return NUQ_EINVAL;
    const uint32_t nsync = nuq_huffman_num_sync(bucket, sync_stride);
    HuffmanCode H;
    if (!huffman_tables(lengths, s, H))
        return NUQ_EINVAL;
    EncodeBatch Wk{};
    for (uint32_t k = 0; k < K; ++k) {
        if (!v[k] || !norms[k] || !bit_off[k] || !words[k] || (nsync && (!sync || !sync[k])) ||
            (reinterpret_cast<uintptr_t>(v[k]) & 3u))
            return NUQ_EINVAL;
        Wk.w[k].v = v[k];
        Wk.w[k].seed = seeds[k];
        Wk.w[k].norms_out = norms[k];
        Wk.w[k].bit_off = bit_off[k];
        Wk.w[k].words = words[k];
        Wk.w[k].words_cap = words_cap[k];
        Wk.w[k].sync = nsync ? sync[k] : nullptr;
    }
    const uint64_t nb = nuq_num_buckets(d, bucket);
    const uint32_t slot_words = huffman_slot_words(bucket, s);
    const Workspace w = carve(workspace, K, nb, slot_words);
    if (w.bytes > workspace_bytes)
        return NUQ_ECAPACITY;
    uint32_t *flags = flags_ptr();
    if (!flags)
        return NUQ_EHIP;
    hipStream_t st = static_cast<hipStream_t>(stream);
    EncodeParams P{};
    P.d = d;
    P.nb = nb;
    P.nb_stride = (nb + 3) & ~3ull;
    P.bucket = bucket;
    P.s = s;
    P.sync_shift = nsync ? log2u(sync_stride) : 0;
    P.nsync = nsync;
    P.slot_words = slot_words;
    P.out_cap = slot_words;
    P.units = w.units;
    P.staging = w.staging;
    P.flags = flags;
    P.stream = stream_loads(d, K);
    const bool narrow = narrow_teams<TeamUse::kHuffman>(nb, K, bucket, s);
    int rc = dispatch_team<TeamUse::kHuffman>(bucket, narrow, [&](auto team_c, auto vpt_c) {
        constexpr int TEAM = decltype(team_c)::value, VPT = decltype(vpt_c)::value;
        using G = TeamGeom<TEAM>;
        P.rows = team_rows<TEAM>(bucket);
        P.lds_words = ((P.rows * TEAM + P.out_cap + nsync + 3u) & ~3u) + 64u;       // 16-byte aligned teams and fields
        const size_t lds_bytes = (size_t)P.lds_words * 4 * G::kTeamsPerWG;
        if (lds_bytes > 160 * 1024)
            return (int)NUQ_EINVAL;
        auto kern = s <= 6u ? k_huffman_fused<TEAM, VPT, true> : k_huffman_fused<TEAM, VPT, false>;
        if (lds_bytes > 48 * 1024 &&
            hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_bytes) != hipSuccess)
            return (int)NUQ_EHIP;
        dim3 grid;
        if (!bucket_grid<TEAM>(nb, K, grid))
            return (int)NUQ_EINVAL;
        ScopedTiming timing(NUQ_T_QUANTIZE_ENCODE, st);
        hipLaunchKernelGGL(kern, grid, dim3(G::kWG), lds_bytes, st, P, Wk, H);
        return check_launch();
    });
    if (rc != NUQ_OK)
        return rc;
    return launch_finish(P, Wk, K, w, narrow, st);
}

int nuq_decode_huffman_batch(uint32_t K, const uint64_t *const *bit_off, const uint32_t *const *words,
                             const uint32_t *const *sync, uint64_t d, uint32_t bucket, uint32_t s,
                             uint32_t sync_stride, const uint8_t *lengths, uint8_t *const *q, nuq_stream_t stream)
{
    if (K < 1 || K > kMaxBatch || !bit_off || !words || !lengths || !q || !valid_common(d, bucket, s) ||
        !valid_sync(sync_stride))
        return NUQ_EINVAL;
    const uint32_t nsync = nuq_huffman_num_sync(bucket, sync_stride);
    if (nsync && !sync)
        return NUQ_EINVAL;
    HuffmanCode H;
    if (!huffman_tables(lengths, s, H))
        return NUQ_EINVAL;
    uint32_t *flags = flags_ptr();
    if (!flags)
        return NUQ_EHIP;
    HuffmanDecodeParams P{};
    for (uint32_t k = 0; k < K; ++k) {
        if (!bit_off[k] || !words[k] || !q[k] || (nsync && !sync[k]))
            return NUQ_EINVAL;
        P.w[k] = HuffmanStream{bit_off[k], words[k], nsync ? sync[k] : nullptr, q[k]};
    }
    P.flags = flags;
    P.d = d;
    P.nb = nuq_num_buckets(d, bucket);
    P.bucket = bucket;
    P.sync_shift = nsync ? log2u(sync_stride) : 0;
    P.nsync = nsync;
    P.nseg = nsync + 1;
    const uint64_t units = P.nb * P.nseg;
    const uint64_t blocks = nsync ? (units + 63) / 64 : (units + 255) / 256;
    if (blocks > 0x7fffffffull)
        return NUQ_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    ScopedTiming timing(NUQ_T_DECODE, st);
    // one staging row per thread: at most 1024 / 16 + 9 words
    const size_t direct_lds = (size_t)kHuffmanDirectWG * huffman_stage_stride(sync_stride) * 4u;
    bool direct = nsync && bucket % 16u == 0 && direct_lds <= 40u * 1024u;
    for (uint32_t k = 0; k < K && direct; ++k)
        direct = (reinterpret_cast<uintptr_t>(q[k]) & 15u) == 0;
    if (direct) {
        const uint64_t wgs = (units + kHuffmanDirectWG - 1) / kHuffmanDirectWG;
        hipLaunchKernelGGL(k_huffman_decode_direct, dim3((uint32_t)wgs, K), dim3(kHuffmanDirectWG), direct_lds, st, P,
                           H);
    } else if (nsync) {
        const size_t lds_bytes = 64u * (sync_stride / 4u + 1u + huffman_stage_stride(sync_stride)) * 4u;
        if (lds_bytes > 48 * 1024 &&
            hipFuncSetAttribute(reinterpret_cast<const void *>(k_huffman_decode_tile),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes) != hipSuccess)
            return NUQ_EHIP;
        hipLaunchKernelGGL(k_huffman_decode_tile, dim3((uint32_t)blocks, K), dim3(64), lds_bytes, st, P, H);
    } else {
        hipLaunchKernelGGL(k_huffman_decode, dim3((uint32_t)blocks, K), dim3(256), 0, st, P, H);
    }
    return check_launch();
}

int nuq_decode_accumulate_huffman(uint32_t K, const float *const *norms, const uint64_t *const *bit_off,
                                  const uint32_t *const *words, const uint64_t *words_len,
                                  const uint32_t *const *sync, uint64_t d, uint32_t bucket, uint32_t s,
                                  uint32_t sync_stride, const uint8_t *lengths, float scale, int accumulate,
                                  float *out, nuq_stream_t stream)
{
    if (K < 1 || K > NUQ_MAX_WORKERS || !norms || !bit_off || !words || !words_len || !sync || !lengths || !out ||
        !valid_common(d, bucket, s) || !valid_sync(sync_stride))
        return NUQ_EINVAL;
    const uint32_t nsync = nuq_huffman_num_sync(bucket, sync_stride);
    HuffmanCode H;
    if (!nsync || !huffman_tables(lengths, s, H))
        return NUQ_EINVAL;
    DecodeParams P{};
    for (uint32_t k = 0; k < K; ++k) {
        if (!norms[k] || !bit_off[k] || !words[k] || !sync[k])
            return NUQ_EINVAL;
        P.norms[k] = norms[k];
        P.bit_off[k] = bit_off[k];
        P.words[k] = words[k];
        P.words_bits[k] = words_len[k] > (UINT64_MAX >> 5) ? UINT64_MAX : words_len[k] << 5;
        P.sync[k] = sync[k];
    }
    P.out = out;
    P.d = d;
    P.nb = nuq_num_buckets(d, bucket);
    P.K = K;
    P.bucket = bucket;
    P.s = s;
    P.scale = scale;
    P.nsync = nsync;
    P.nseg = nsync + 1u;                        // pieces per bucket: ceil(bucket / sync_stride)
    P.sync_shift = log2u(sync_stride);
    P.pieces_shift = log2u(kTileCoords / sync_stride);
    // tiles as for the ERC strings: several whole buckets, or 2048 coordinates of one
    uint64_t ntiles;
    uint32_t max_streams;
    if (bucket <= kTileCoords) {
        const uint32_t by_size = kTileCoords / bucket, by_streams = kMaxStreams / K;
        P.buckets_per_tile = by_size < by_streams ? by_size : by_streams;
        P.tiles_per_bucket = 1;
        P.tile_coords = P.buckets_per_tile * bucket;
        P.segs_per_tile = P.nseg;
        ntiles = (P.nb + P.buckets_per_tile - 1) / P.buckets_per_tile;
        max_streams = P.buckets_per_tile * K;
    } else {
        P.buckets_per_tile = 0;
        P.tile_coords = kTileCoords;
        P.tiles_per_bucket = (bucket + kTileCoords - 1) / kTileCoords;
        P.segs_per_tile = kTileCoords >> P.sync_shift;
        ntiles = P.nb * P.tiles_per_bucket;
        max_streams = K;
    }
    if (ntiles > 0x7fffffffull)
        return NUQ_EINVAL;
    P.ntiles = (uint32_t)ntiles;
    P.xcd_base = P.ntiles / 8u;
    P.xcd_rem = P.ntiles % 8u;
    while ((2u << P.lanes_shift) * max_streams <= 64u)
        ++P.lanes_shift;
    // the lanes that copy a stream's words parse its pieces: a piece per lane
    if (P.segs_per_tile > (1u << P.lanes_shift))
        return NUQ_EINVAL;
    P.parts_shift = P.lanes_shift - log2u(P.segs_per_tile);
    uint32_t *flags = flags_ptr();
    if (!flags)
        return NUQ_EHIP;
    P.flags = flags;
    auto kern = accumulate ? k_decode_wave_huffman<kUpdateAdd> : k_decode_wave_huffman<kUpdateWrite>;
    static uint32_t cached[2][64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return NUQ_EHIP;
    uint32_t &resident = cached[accumulate ? 1 : 0][dev];
    if (!resident) {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kern), (int)kWaveWG,
                                                         0) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || per_cu < 1 ||
            cus < 1)
            return NUQ_EHIP;
        resident = ((uint32_t)per_cu * (uint32_t)cus) & ~7u;          // a multiple of the eight XCDs (see xcd_tile)
        if (!resident)
            resident = 8u;
    }
    const uint32_t grid = P.ntiles < resident ? P.ntiles : resident;
    ScopedTiming timing(NUQ_T_DECODE, static_cast<hipStream_t>(stream));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kWaveWG), 0, static_cast<hipStream_t>(stream), P, H);
    return check_launch();
}

int nuq_decode_huffman(const uint64_t *bit_off, const uint32_t *words, const uint32_t *sync, uint64_t d,
                       uint32_t bucket, uint32_t s, uint32_t sync_stride, const uint8_t *lengths, uint8_t *q,
                       nuq_stream_t stream)
{
    return nuq_decode_huffman_batch(1, &bit_off, &words, &sync, d, bucket, s, sync_stride, lengths, &q, stream);
}

int nuq_average_levels(uint32_t K, const float *const *norms, const uint8_t *const *q, uint64_t d, uint32_t bucket,
                       uint32_t s, float scale, int accumulate, float *out, nuq_stream_t stream)
{
    if (K < 1 || K > NUQ_MAX_WORKERS || !norms || !q || !out || !valid_common(d, bucket, s))
        return NUQ_EINVAL;
    AverageParams P{};
    bool aligned = bucket % 4u == 0;
    for (uint32_t k = 0; k < K; ++k) {
        if (!norms[k] || !q[k])
            return NUQ_EINVAL;
        P.norms[k] = norms[k];
        P.q[k] = q[k];
        aligned = aligned && (reinterpret_cast<uintptr_t>(q[k]) & 3u) == 0;
    }
    P.out = out;
    P.d = d;
    P.K = K;
    P.bucket = bucket;
    P.s = s;
    P.scale = scale;
    P.accumulate = accumulate;
    bool wide = aligned && bucket % 16u == 0 && (reinterpret_cast<uintptr_t>(out) & 15u) == 0;
    for (uint32_t k = 0; k < K && wide; ++k)
        wide = (reinterpret_cast<uintptr_t>(q[k]) & 15u) == 0;
    const uint64_t threads = wide ? (d + 15) / 16 : aligned ? (d + 3) / 4 : d, blocks = (threads + 255) / 256;
    if (blocks > 0x7fffffffull)
        return NUQ_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (wide) {
        // value tables in LDS when those of the buckets a workgroup (4096 coordinates) can touch fit in 16 KB
        const uint64_t nb = nuq_num_buckets(d, bucket);
        const bool tiled = 4096u % bucket == 0 || bucket % 4096u == 0;
        const uint64_t tabs = std::min<uint64_t>(nb, tiled ? std::max(1u, 4096u / bucket) : 4096u / bucket + 2u);
        const uint64_t lut_bytes = tabs * K * 32u * sizeof(double);
        P.lut_tabs = (uint32_t)tabs;
        if (lut_bytes <= 16384u)
            hipLaunchKernelGGL(k_average_levels16<true>, dim3((uint32_t)blocks), dim3(256), (uint32_t)lut_bytes, st, P);
        else
            hipLaunchKernelGGL(k_average_levels16<false>, dim3((uint32_t)blocks), dim3(256), 0, st, P);
    }
    else if (aligned)
        hipLaunchKernelGGL(k_average_levels<4>, dim3((uint32_t)blocks), dim3(256), 0, st, P);
    else
        hipLaunchKernelGGL(k_average_levels<1>, dim3((uint32_t)blocks), dim3(256), 0, st, P);
    return check_launch();
}

int nuq_momentum_step(float *w, float *yl, const float *g, uint64_t d, float alpha, float mu, float l,
                      nuq_stream_t stream)
{
    if (!std::isfinite(alpha) || !std::isfinite(mu) || !std::isfinite(l) || mu < 0.0f || !(mu < 1.0f))
        return NUQ_EINVAL;
    if (d == 0)
        return NUQ_OK;
    if (!w || !yl || !g)
        return NUQ_EINVAL;
    const bool vec = ((reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(yl) |
                       reinterpret_cast<uintptr_t>(g)) & 15u) == 0;
    const uint64_t threads = vec ? (d + 3) / 4 : d, blocks = (threads + 255) / 256;
    if (blocks > 0x7fffffffull)
        return NUQ_EINVAL;
    const MomentumParams P{w, yl, g, d, (double)alpha, (double)mu, (double)l};
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (vec)
        hipLaunchKernelGGL(k_momentum_step<true>, dim3((uint32_t)blocks), dim3(256), 0, st, P);
    else
        hipLaunchKernelGGL(k_momentum_step<false>, dim3((uint32_t)blocks), dim3(256), 0, st, P);
    return check_launch();
}

int nuq_decode_momentum_step(uint32_t K, const float *const *norms, const uint64_t *const *bit_off,
                             const uint32_t *const *words, const uint64_t *words_len,
                             const uint32_t *const *sync, uint64_t d, uint32_t bucket, uint32_t s,
                             uint32_t sync_stride, float scale, float alpha, float mu, float l, float *w, float *yl,
                             nuq_stream_t stream)
{
    if (!std::isfinite(alpha) || !std::isfinite(mu) || !std::isfinite(l) || mu < 0.0f || !(mu < 1.0f) || !yl)
        return NUQ_EINVAL;
    const MomentumParams M{w, yl, nullptr, d, (double)alpha, (double)mu, (double)l};
    return decode_accumulate_any(K, norms, bit_off, words, words_len, sync, d, bucket, s, sync_stride, nullptr, scale,
                                 0, w, stream, &M);
}

int nuq_moments_accumulate(const float *g, double *sum, double *sumsq, uint64_t d, nuq_stream_t stream)
{
    if (d == 0)
        return NUQ_OK;
    if (!g || !sum || !sumsq)
        return NUQ_EINVAL;
    const bool vec = (reinterpret_cast<uintptr_t>(g) & 7u) == 0 &&
                     ((reinterpret_cast<uintptr_t>(sum) | reinterpret_cast<uintptr_t>(sumsq)) & 15u) == 0;
    const uint64_t threads = vec ? (d + 1) / 2 : d, blocks = (threads + 255) / 256;
    if (blocks > 0x7fffffffull)
        return NUQ_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (vec)
        hipLaunchKernelGGL(k_moments_accumulate<true>, dim3((uint32_t)blocks), dim3(256), 0, st, g, sum, sumsq, d);
    else
        hipLaunchKernelGGL(k_moments_accumulate<false>, dim3((uint32_t)blocks), dim3(256), 0, st, g, sum, sumsq, d);
    return check_launch();
}

int nuq_normalized_variance(const double *sum, const double *sumsq, uint64_t d, uint64_t M, void *workspace,
                            uint64_t workspace_bytes, double *out2, nuq_stream_t stream)
{
    static_assert(NUQ_VARIANCE_WORKSPACE_BYTES == kVarianceBlocks * 2u * sizeof(double), "workspace size");
    if (M < 1 || !out2 || !workspace || workspace_bytes < NUQ_VARIANCE_WORKSPACE_BYTES ||
        (reinterpret_cast<uintptr_t>(workspace) & 7u) != 0 || (d > 0 && (!sum || !sumsq)))
        return NUQ_EINVAL;
    double *partial = static_cast<double *>(workspace);
    const uint32_t blocks = (uint32_t)std::min<uint64_t>(kVarianceBlocks, std::max<uint64_t>(1, (d + 255) / 256));
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_variance_partials, dim3(blocks), dim3(256), 0, st, sum, sumsq, d, 1.0 / (double)M, partial);
    hipLaunchKernelGGL(k_variance_finish, dim3(1), dim3(256), 0, st, partial, blocks, out2);
    return check_launch();
}

int nuq_last_error_flags(uint32_t *host_flags, nuq_stream_t stream)
{
    if (!host_flags)
        return NUQ_EINVAL;
    uint32_t *flags = flags_ptr();
    if (!flags)
        return NUQ_EHIP;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (hipMemcpyAsync(host_flags, flags, sizeof(uint32_t), hipMemcpyDeviceToHost, st) != hipSuccess)
        return NUQ_EHIP;
    if (hipStreamSynchronize(st) != hipSuccess)
        return NUQ_EHIP;
    const uint32_t zero = 0;
    if (hipMemcpyAsync(flags, &zero, sizeof(uint32_t), hipMemcpyHostToDevice, st) != hipSuccess)
        return NUQ_EHIP;
    if (hipStreamSynchronize(st) != hipSuccess)
        return NUQ_EHIP;
    return NUQ_OK;
}

int nuq_encode_shape(uint32_t mode, uint32_t K, uint64_t d, uint32_t bucket, uint32_t s, uint32_t sync_stride,
                     const float *levels, uint32_t norm_kind, uint32_t *shape)
{
    if (mode > 2 || K < 1 || K > kMaxBatch || !valid_common(d, bucket, s) || !valid_sync(sync_stride) || !shape ||
        (mode == 2 && (!levels || !valid_levels(levels, s))))
        return NUQ_EINVAL;
    EncodeParams P{};
    bool narrow;
    auto tell = [&](auto team_c, auto, const TeamLdsMap &map) {
        constexpr int TEAM = decltype(team_c)::value;
        shape[0] = TEAM;
        shape[1] = P.rec_cap;
        shape[2] = P.out_cap;
        shape[3] = map.sync - map.rec;
        return (int)NUQ_OK;
    };
    const double l1 = mode == 2 ? (double)levels[1] : std::ldexp(1.0, -(int)s);
    const bool linf = mode == 2 && norm_kind == NUQ_NORM_LINF;
    return mode == 0   ? with_encode_shape<0>(P, K, d, bucket, s, sync_stride, l1, linf, narrow, tell)
           : mode == 1 ? with_encode_shape<1>(P, K, d, bucket, s, sync_stride, l1, linf, narrow, tell)
                       : with_encode_shape<2>(P, K, d, bucket, s, sync_stride, l1, linf, narrow, tell);
}

uint32_t nuq_decode_tile(uint32_t K, uint64_t d, uint32_t bucket, uint32_t s, uint32_t sync_stride, int table, uint32_t update)
{
    if (K < 1 || K > NUQ_MAX_WORKERS || !valid_common(d, bucket, s) || !valid_sync(sync_stride))
        return 0;
    return decode_tile_coords(K, d, bucket, s, sync_stride, table != 0, update);
}

int nuq_timing_begin(uint32_t max_launches)
{
    if (max_launches > 4096 || g_timing.cap != 0)
        return NUQ_EINVAL;
    g_timing.start.resize(max_launches);
    g_timing.stop.resize(max_launches);
    g_timing.entry.assign(max_launches, 0);
    for (uint32_t i = 0; i < max_launches; ++i)
        if (hipEventCreate(&g_timing.start[i]) != hipSuccess || hipEventCreate(&g_timing.stop[i]) != hipSuccess)
            return NUQ_EHIP;
    g_timing.used = 0;
    g_timing.cap = max_launches;
    return NUQ_OK;
}

int nuq_timing_collect(float *ms, int32_t *entry, uint32_t cap, uint32_t *count)
{
    if (!ms || !entry || !count)
        return NUQ_EINVAL;
    int rc = NUQ_OK;
    uint32_t n = 0;
    for (uint32_t i = 0; i < g_timing.used; ++i) {
        if (hipEventSynchronize(g_timing.stop[i]) != hipSuccess)
            rc = NUQ_EHIP;
        float t = 0.f;
        if (hipEventElapsedTime(&t, g_timing.start[i], g_timing.stop[i]) != hipSuccess)
            rc = NUQ_EHIP;
        if (n < cap) {
            ms[n] = t;
            entry[n] = g_timing.entry[i];
            ++n;
        }
    }
    for (uint32_t i = 0; i < g_timing.cap; ++i) {
        (void)hipEventDestroy(g_timing.start[i]);
        (void)hipEventDestroy(g_timing.stop[i]);
    }
    g_timing = Timing{};
    *count = n;
    return rc;
}

}  // extern "C"
