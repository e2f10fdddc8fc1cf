/*
 * Measurement aids of the CSB-RNN library (csbrnn.h).  NOT operations of the method and not
 * part of the stable interface: bench.py and the tests use them to produce the load-balance and
 * bandwidth figures that are reported next to the kernels' timings.  Same conventions as
 * csbrnn.h (device pointers, 0 on success, csb_last_error()).
 */
#ifndef CSBRNN_DEBUG_H
#define CSBRNN_DEBUG_H

#include "csbrnn.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * csb_spmv with clock stamps, for load-balance evidence: same result, and every wavefront also
 * writes stamps to d_stamps (device, csb_debug_stamp_count(m) values of 64 bits).
 * Row-owned layout: per workgroup and wavefront 8 values of the 100 MHz wall clock: start, input
 * vector staged (after the barrier), first segment unit in LDS (twice), products done, after
 * the last barrier, end, one unused.  Tile-based layout: per workgroup 8 phase stamps of the
 * shader clock (start, loads issued, staged in LDS, mat-vec done, tile sums written, end, 2
 * unused), then three for each of its 16 wavefronts: begin of its share, its kernel values
 * arrived, end of the share.  d_ws as for csb_spmv.
 */
size_t csb_debug_stamp_count(const csb_matrix *m);
int csb_debug_spmv_stamps(const csb_matrix *m, const float *d_x, float *d_y, void *d_ws,
                          unsigned long long *d_stamps, void *stream);

/*
 * A plain streaming read of d_buf (device, 16-byte aligned, `bytes` a multiple of 16) whose
 * timing gives the read bandwidth this GPU reaches in practice for a launch of that size.
 * Every thread writes its partial sum to d_out (device, csb_debug_stream_read_out_floats()
 * floats).  Asynchronous on `stream`.
 */
size_t csb_debug_stream_read_out_floats(void);
int csb_debug_stream_read(const void *d_buf, size_t bytes, float *d_out, void *stream);

/*
 * Right-hand sides per workgroup (64 or 128) that csb_spmm (bits16 = 0) and csb_spmm_bfloat / csb_spmm_half
 * (bits16 = 1) choose on a plan of `row_tiles` row tiles of 16 or 32 rows, where the form that keeps
 * its results in registers runs.  Host only.
 */
int csb_debug_spmm_columns(int64_t row_tiles, int32_t rows_per_tile, int32_t batch, int32_t bits16);

/*
 * Passes (at most 8 columns by the rows of one block in one row tile) of the section that the batched products read, in row
 * tiles of 16 or 32 rows; 0 where the plan has no such section.  Host only.
 */
int64_t csb_debug_quad_passes(const csb_matrix *m, int32_t rows_per_tile);

/*
 * What the batched products of `m` read: 0 (the default): what an estimate of the launch's time favours; 1: the tile-based
 * sections; 2: the section of four-row steps wherever it can be read.  16-bit values times 16-bit right-hand sides read that
 * section, in panels of eight columns, unless the tile-based ones are asked for.
 */
int csb_debug_spmm_force(csb_matrix *m, int32_t form);

/*
 * The form that csb_spmm (bits16 = 0) or csb_spmm_bfloat / csb_spmm_half (bits16 = 1: csb_debug_spmm_panel's answer) takes for
 * `batch` contiguous right-hand sides:
 * form[0] = rows of a tile of the section of four-row steps (0: the tile-based sections), form[1] = right-hand sides and
 * form[2] = wavefronts of a workgroup.  Host only.
 */
int csb_debug_spmm_form(const csb_matrix *m, int32_t batch, int32_t bits16, int32_t *form);
/* The same for the panels of csb_spmm_bfloat / csb_spmm_half (form[0] = 0: the call takes none). */
int csb_debug_spmm_panel(const csb_matrix *m, int32_t batch, int32_t *form);

/*
 * Whether csb_rnn_forward runs a batch on the resident kernel (1) or on the batched products (0) when the layouts
 * of both are uploaded.  Host only.
 */
int csb_debug_rnn_prefers_resident(const csb_rnn *rnn, int32_t batch);

#ifdef __cplusplus
}
#endif

#endif
