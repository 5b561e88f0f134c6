/*
 * libwinof4 measurement probes -- not part of the convolution and not part of
 * the method's interface.  They are exported by the same library so that a
 * benchmark can state the int8 matrix-core rate it measures at the run's
 * clock next to the datasheet figure, the denominator a tap-GEMM utilisation
 * is read against, and so that a benchmark or a test can tell which kernels a
 * convolution launches.
 */
#ifndef WINOF4_PROBE_H
#define WINOF4_PROBE_H

#include "winof4.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * wino_probe_mfma_int8 -- measurement probe, not part of the convolution:
 * `blocks` workgroups of four waves issue independent int8 MFMAs only
 * (shape 16: v_mfma_i32_16x16x64_i8, eight chains per wave; shape 32:
 * v_mfma_i32_32x32x32_i8, four chains), `iters` rounds each, so that a
 * caller timing the launch measures the int8 matrix-core rate at the run's
 * clock.  *ops (host) receives the launch's operation count (2 per
 * multiply-add).  sink: device int32, never written in practice (it keeps
 * the results live).  Asynchronous on `stream`; WINO_EINVAL for a bad shape
 * or count or a NULL pointer.
 */
wino_status wino_probe_mfma_int8(int32_t shape, int32_t iters, int32_t blocks, int32_t* sink,
                                 int64_t* ops, hipStream_t stream);

/*
 * wino_probe_conv_kernels -- the kernels that a SPLIT wino_f4_conv_int8 with
 * this plan launches for an n x h x w input x (only its address is looked at),
 * an output apart from it and a workspace of wino_f4_workspace_bytes.  Host only, no device work.
 * All fields are 0 for an empty input.  Errors: WINO_EINVAL (null plan or k,
 * negative sizes, unknown layout), WINO_EUNSUPPORTED (sizes beyond the
 * library's limits).
 */
enum { WINO_PROBE_XFORM_NONE = 0,      /* part of the one launch                    */
       WINO_PROBE_XFORM_DIRECT = 1,    /* NHWC, pixels straight to registers        */
       WINO_PROBE_XFORM_BAND = 2 };    /* through a halo band in LDS                */
enum { WINO_PROBE_GEMM_SMALL = 1,      /* one wave per row of taps                  */
       WINO_PROBE_GEMM_RESIDENT = 2,   /* all taps of a block in registers          */
       WINO_PROBE_GEMM_ROWS = 3,       /* row-streamed, int8                        */
       WINO_PROBE_GEMM_ROWS_STREAMK = 4,
       WINO_PROBE_GEMM_WAVES = 5,      /* wave-specialized                          */
       WINO_PROBE_GEMM_ROWS_WIDE = 6 };/* row-streamed, int8/10                     */
typedef struct wino_probe_kernels {
    int32_t launches;                  /* 1: the whole convolution in one launch    */
    int32_t xform, xform_tiles;        /* input transform, its tiles per block      */
    int32_t gemm, co, tiles;           /* tap GEMM, its block: channels x tiles     */
} wino_probe_kernels;
wino_status wino_probe_conv_kernels(wino_f4_plan_t plan, const int8_t* x, int32_t n, int32_t h, int32_t w,
                                    wino_layout layout, wino_probe_kernels* k);

#ifdef __cplusplus
}
#endif

#endif /* WINOF4_PROBE_H */
