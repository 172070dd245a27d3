/*
 * adatopk_measure.h -- measurement hooks of libadatopk (benchmarks, profiling and tests only).
 *
 * Not part of the compressor's contract: these calls exist so that a benchmark can
 * time the individual kernels of a compress / decompress call with HIP events on the
 * caller's stream, and can measure plain streaming kernels (the ceilings that the
 * HBM roofline fractions are compared with, and the known-size copy that hardware
 * counter readings are scaled by).  They keep process-global state, create HIP events
 * and synchronise; none of them may be used concurrently with another call.
 */
#ifndef ADATOPK_MEASURE_H
#define ADATOPK_MEASURE_H

#include <stddef.h>
#include <stdint.h>

#include "adatopk.h"

#ifdef __cplusplus
extern "C" {
#endif

/* on != 0: from now on every kernel of a compress / decompress call is launched with a
 * start and a stop HIP event that carry the timestamps of the dispatch itself (events are
 * created as they are needed).  on == 0: plain launches.  Returns ADATOPK_OK or
 * ADATOPK_ERUNTIME. */
adatopk_status adatopk_measure_enable(int32_t on);

/* Number of kernel stages a timed call can report, and their names (static strings):
 * the kernels of compress in launch order, then those of the two decompress calls. */
int32_t adatopk_measure_stage_count(void);
const char *adatopk_measure_stage_name(int32_t stage);

/* Waits for the stop events of the kernels launched since the last read and stores the
 * summed duration of the launches of every stage (a batch is launched in groups; the first 64 of
 * a stage count) in milliseconds into
 * ms_out[adatopk_measure_stage_count()] (host memory); stages that did not run since
 * the last read are reported as -1.  Returns ADATOPK_OK or ADATOPK_ERUNTIME. */
adatopk_status adatopk_measure_read(float *ms_out);

/* For tests of the compress of a single tensor whose sample misled it: from now on the kernel that then makes
 * the exact passes is launched without its last `missing_workgroups` workgroups, as if they started too late;
 * those that are there do their chunks for them.  Wrong results for a tensor whose sample did not mislead.
 * 0: all workgroups.  wait_rounds: how often a workgroup looks for the others before it gives up (the call then
 * ends with a NaN error norm); negative: as in the product library. */
void adatopk_measure_judge(int32_t missing_workgroups, int32_t wait_rounds);

/* Byte offset in the workspace of a call over `n_total` elements of
 *   ADATOPK_MEASURE_CLAIMS        (a single tensor whose sample misled it) who worked: per chunk 1 + the number of the
 *                                 workgroup that took it, 0 if none had to (uint32)
 *   ADATOPK_MEASURE_CHUNK_COUNTS  per chunk its candidates, more than a quarter of the chunk's length: the chunk
 *                                 has no list (uint32)
 *   ADATOPK_MEASURE_PART_COUNTS   (fp32) per part of a chunk's candidates how many lie above the k-th key's window bin; not
 *                                 written for empty parts (uint32) */
#define ADATOPK_MEASURE_CLAIMS 0
#define ADATOPK_MEASURE_CHUNK_COUNTS 1
#define ADATOPK_MEASURE_PART_COUNTS 2
size_t adatopk_measure_workspace_offset(int32_t what, int64_t n_total, int32_t num_segments, adatopk_dtype dtype);

/* Plain streaming kernels on `hip_stream`; all pointers are device memory, 16-byte
 * aligned; bytes must be a multiple of 16.
 *   copy:      dst[i] = src[i]                        (reads bytes, writes bytes)
 *   read_only: folds src into one word at sink[0]     (reads bytes)
 *   fill:      dst[i] = 0, the kernel decompress uses (writes bytes) */
adatopk_status adatopk_measure_copy(void *dst, const void *src, size_t bytes, void *hip_stream);
adatopk_status adatopk_measure_read_only(const void *src, size_t bytes, uint32_t *sink, void *hip_stream);
adatopk_status adatopk_measure_fill(void *dst, size_t bytes, void *hip_stream);

#ifdef __cplusplus
}
#endif
#endif /* ADATOPK_MEASURE_H */
