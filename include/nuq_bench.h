/* Measurement aids of libnuq.so: per-launch kernel times for benchmarks, launch shapes for tests.
 *
 * Not part of the method and not needed by a caller of include/nuq.h: bench.py brackets the main kernel
 * of each entry point with HIP events on the stream the kernel is launched on (the capture is
 * process-global state: one capture at a time, not thread-safe), and the tests ask where the lines of a
 * launch rule lie, so that their inputs stay on both sides of them.
 */
#ifndef NUQ_BENCH_H
#define NUQ_BENCH_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* Entry-point ids reported by nuq_timing_collect. */
enum { NUQ_T_NORMS = 1, NUQ_T_QUANTIZE = 2, NUQ_T_ENCODE = 3, NUQ_T_QUANTIZE_ENCODE = 4, NUQ_T_DECODE = 5 };

/* After nuq_timing_begin(n), each of the next n launches of a main kernel (the per-bucket kernel
 * of nuq_bucket_norms / nuq_quantize / nuq_encode / nuq_quantize_encode, the tile kernel of
 * nuq_decode_accumulate) is bracketed by a pair of HIP events recorded on its stream.  The small
 * offset-scan and gather kernels of the encoders are outside the brackets.  n <= 4096.
 * Not thread-safe; meant for benchmarks. */
int nuq_timing_begin(uint32_t max_launches);

/* Waits for the bracketed launches, writes up to `cap` durations (milliseconds) and entry-point
 * ids to the HOST arrays ms[] and entry[], the number written to *count, and ends the capture. */
int nuq_timing_collect(float *ms, int32_t *entry, uint32_t cap, uint32_t *count);

/* How the main kernel of the ERC encoders is laid out for a call of these sizes (host arithmetic).  mode 0:
 * nuq_quantize_encode(_batch), 1: nuq_encode, 2: nuq_quantize_encode_table_batch (levels, norm_kind as
 * there, HOST memory; ignored in the others).  shape (HOST, 4 values): threads per bucket; nonzeros that
 * a bucket's list in LDS holds; words of its bit string that the string's buffer holds; words of the
 * string of a bucket whose nonzeros do not fit the list that are put together at once. */
int nuq_encode_shape(uint32_t mode, uint32_t K, uint64_t d, uint32_t bucket, uint32_t s,
                     uint32_t sync_stride, const float *levels, uint32_t norm_kind, uint32_t *shape);

/* Coordinates of a tile of the decoder for K messages of these sizes (where it works in tiles), 0 on invalid
 * sizes.  table: levels from a table; update: 0 = the result is written, 1 = added, 2 = momentum rule. */
uint32_t nuq_decode_tile(uint32_t K, uint64_t d, uint32_t bucket, uint32_t s, uint32_t sync_stride, int table,
                         uint32_t update);

#ifdef __cplusplus
}
#endif
#endif /* NUQ_BENCH_H */
