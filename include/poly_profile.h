/*
 * libpoly measurement hooks -- NOT part of the method and outside the "allocates nothing" contract of poly.h:
 * poly_profile_begin creates host-side HIP events for the launches it records.
 */
#ifndef POLY_PROFILE_H
#define POLY_PROFILE_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* Per-stage kernel timing for measurement harnesses.  Between
 * poly_profile_begin and poly_profile_end every kernel the library launches carries a start/stop
 * event pair stamped by the runtime with the dispatch's own begin and end, and poly_profile_end
 * (which synchronises the device) returns, per stage, the number of launches and the sum of their
 * execution times in milliseconds.  `max_launches` bounds the number of recorded launches (host
 * events are created for them); launches beyond it run untimed.  Process-wide, not thread-safe.
 */
enum {
    POLY_STAGE_SELECT = 0, /* Alg. 2 kernel */
    POLY_STAGE_GEMM = 1,   /* base linears with fused expand and epilogue (patch embedding included), and launches that hold more: the
                              row kernels (LayerNorm and shrink too), the task queues (a run of whole layers: attention, LayerNorm and
                              shrink too), the patch embedding of frames that its product gathers itself (with the class token and the CSR
                              check), LayerNorm + linear of few frames of a wide model, and the isolated linear of a small call (CSR
                              check and shrink too) */
    POLY_STAGE_SHRINK = 2, /* x A_k, where it is a launch of its own (of the isolated bf16 linear: with the CSR check) */
    POLY_STAGE_ATTN = 3,   /* where it is a launch of its own */
    POLY_STAGE_NORM = 4,   /* LayerNorm, likewise; of a wide model with adapters: with the shrink of its rows */
    POLY_STAGE_OTHER = 5,  /* CSR check, patch gathering and class token, likewise; heads, merge */
    POLY_STAGE_COUNT = 6
};

typedef struct poly_profile {
    int32_t launches[POLY_STAGE_COUNT];
    float ms[POLY_STAGE_COUNT];
    int32_t dropped; /* recorded launches whose events could not be read */
} poly_profile;

int poly_profile_begin(int max_launches);
int poly_profile_end(poly_profile *out); /* host struct */

/* How often a workgroup of a kernel that runs many layers in one launch may look at a counter that is not there yet, in calls of the calling thread from
 * now on; negative = the built-in limit (the default).  For tests of what a call does when such a kernel gives up (POLY_ESTALL).  (Of the tiles that stay on
 * their CUs the wait for a block's workgroups to be there has this limit where it is below the built-in one, and else one of its own, of half a minute.) */
void poly_wait_limit(int looks);

/* Workgroups of a launch of the wide models' task queue, or of tiles that stay on their CUs, at most, in calls of the calling thread from now on; 0 = one per
 * CU (the default).  For tests of their progress with fewer workgroups than queues. */
void poly_wait_workgroups(int most);

#ifdef __cplusplus
}
#endif
#endif /* POLY_PROFILE_H */
