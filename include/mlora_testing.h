/*
 * mlora_testing.h -- test and measurement switches of libmlora.
 *
 * Not part of the operator's interface (mlora.h): a process-wide switch that forces the general
 * kernels, so that tests can compare every kernel mix on one shape, and a timing aid that
 * brackets the library's kernel launches with HIP events.  Unlike the entry points of mlora.h
 * the timing aid allocates: it creates HIP events (hipEventCreate) on first use and keeps them
 * until the process ends.  Production callers need neither.
 */
#ifndef MLORA_TESTING_H
#define MLORA_TESTING_H

#include "mlora.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Selects which kernels the entry points use (bit mask):
 *   0 (default) fastest applicable path: aligned bf16 kernels (with forms of their own for ranks
 *               that are no multiple of 8) when the problem is bf16, h and d are multiples of 64 (the base
 *               products: of 8) and all buffers are 16-byte aligned; the general kernels otherwise,
 *   bit 0       general kernels for the two base products,
 *   bit 1       general kernels for the low-rank products (3 = general everywhere).
 * Returns the previous value.  Process-wide. */
int mlora_set_kernel_path(int path);

/* How the launches of a forward and a backward call of `p` are cut up (plain calls on 16-byte aligned
 * buffers; honours mlora_set_kernel_path), so that a test can hold the sizes it uses to the forms it
 * means to run.  Looks at sizes and addresses only and launches nothing.  `plan` (HOST,
 * MLORA_PLAN_FIELDS entries) is written when `p` is valid; returns the status of mlora_lora_validate. */
#define MLORA_PLAN_Y        0  /* form of the base product of Y: an MLORA_FORM_*                   */
#define MLORA_PLAN_Y_PARTS  1  /* ... contraction ranges per tile                                  */
#define MLORA_PLAN_DX       2  /* the same for dX                                                  */
#define MLORA_PLAN_DX_PARTS 3
#define MLORA_PLAN_Z_ROWS   4  /* s x A: rows per block                                            */
#define MLORA_PLAN_Z_PARTS  5  /* ... contraction ranges                                           */
#define MLORA_PLAN_G_ROWS   6  /* the same for s dy B^T                                            */
#define MLORA_PLAN_G_PARTS  7
#define MLORA_PLAN_GRADS    8  /* dA, dB of a call that wants dX: token ranges per task             */
#define MLORA_PLAN_FIELDS   9
#define MLORA_FORM_WHOLE    0  /* aligned: 256 x 256 tiles                                         */
#define MLORA_FORM_HALVES   1  /* aligned: 128 x 256 tiles                                         */
#define MLORA_FORM_MIXED    2  /* aligned: whole rounds of the first, the rest as the second       */
#define MLORA_FORM_SKINNY   3  /* general: 16 x 64 (aligned problems of few tiles too)             */
#define MLORA_FORM_64       4  /* general: 64 x 64                                                 */
#define MLORA_FORM_128      5  /* general: 128 x 128; the tiles beyond whole rounds of 256 may run as
                                  quarters of 64 x 64, in the ranges that *_PARTS gives            */
#define MLORA_FORM_RING     6  /* aligned: 64 x 64 tiles from a ring                               */
mlora_status mlora_kernel_plan(const mlora_problem* p, int32_t* plan);

/* The tiles of the two base products in the size that their form names (256 x 256 for WHOLE, HALVES and
 * MIXED): how many run as such, and how many there are -- the others run as halves (HALVES, MIXED) or
 * quarters (128); and the rows of the smallest tiles that run: 256, 128, 64 or 16.  And whether a call
 * that wants dX runs it and the gradients in one launch (then the ranges of dX and of the gradients are
 * those of that launch), and the token ranges of dA, dB without dX.  `tiles` (HOST, MLORA_PLAN_TILES
 * entries) and the status as for mlora_kernel_plan. */
#define MLORA_PLAN_Y_WHOLE  0
#define MLORA_PLAN_Y_TILES  1
#define MLORA_PLAN_DX_WHOLE 2
#define MLORA_PLAN_DX_TILES 3
#define MLORA_PLAN_Y_ROWS   4
#define MLORA_PLAN_DX_ROWS  5
#define MLORA_PLAN_SHARED   6
#define MLORA_PLAN_GRADS_ALONE 7
#define MLORA_PLAN_TILES    8
mlora_status mlora_kernel_plan_tiles(const mlora_problem* p, int32_t* tiles);

/* The same for the summed input gradient of a group (`plan`: HOST, MLORA_PLAN_GROUP entries); returns the
 * status of mlora_lora_group_validate. */
#define MLORA_PLAN_GROUP_DX       0  /* form: an MLORA_FORM_*                                      */
#define MLORA_PLAN_GROUP_DX_PARTS 1  /* contraction ranges per tile, over all projections          */
#define MLORA_PLAN_GROUP_DX_WHOLE 2  /* tiles that run as such                                     */
#define MLORA_PLAN_GROUP_DX_TILES 3  /* tiles                                                      */
#define MLORA_PLAN_GROUP_DX_ROWS  4  /* rows of the smallest tiles                                 */
#define MLORA_PLAN_GROUP          5
mlora_status mlora_kernel_plan_group(const mlora_problem* const* ps, int P, int32_t* plan);

/* Measurement aid.  While enabled, every launch of the MFMA kernels by this process, reductions
 * of their ranges included, is bracketed by a pair of HIP events recorded on the launch stream
 * (at most 16384 launches are kept; the events are created on first use and live until the
 * process ends).  Returns the previous setting. */
int mlora_profile_kernels(int enable);

/* Kinds of kernels the measurement aid tells apart, and the unit their work is counted in. */
#define MLORA_PROFILE_GEMM  0  /* base products with their LoRA steps; algorithmic flops
                                  (2 M N K plus 2 t_k r_k N per task).  The input gradient of a
                                  small call runs in one launch with dA_k and dB_k, which are
                                  counted here then, 2 t_k r_k (h + d) per task                */
#define MLORA_PROFILE_ROWS  1  /* s x A and s dy B^T; algorithmic bytes (activation rows read
                                  once, result written once, adapter matrices read once)       */
#define MLORA_PROFILE_GRAD  2  /* dA_k and dB_k; algorithmic bytes                             */
#define MLORA_PROFILE_KINDS 3

/* Waits for the recorded launches to finish; for each kind returns the sum of their durations
 * in milliseconds, the sum of their work in that kind's unit, and their count, through the
 * non-NULL pointers (HOST arrays of MLORA_PROFILE_KINDS entries), and forgets them. */
mlora_status mlora_profile_kernels_read(double* ms_total, double* units_total, int* launches);

#ifdef __cplusplus
}
#endif
#endif /* MLORA_TESTING_H */
