/*
 * eb_route.h -- which kernel a pooled lookup takes.
 *
 * For tests and measurements: it is not part of the pooled-lookup path
 * (include/eb.h), runs on the host and touches no device.
 */
#ifndef EB_ROUTE_H
#define EB_ROUTE_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

enum { EB_ROUTE_PLAIN = 0, EB_ROUTE_TEAM = 1, EB_ROUTE_WAVE = 2 };

/* One eb_forward / eb_forward_ex call, as the choice of its kernel sees it. */
typedef struct eb_route_call {
    int32_t D, dtype, mode;
    int32_t table_align;   /* largest power of two up to 16 dividing every table pointer, */
    int32_t out_align;     /* every output row start in bytes, */
    int32_t offsets_align; /* and the offsets pointer */
    int64_t T, B, nnz;
    int64_t table_rows;    /* rows of every table, */
    int64_t local_rows;    /* and how many of them can be gathered here */
} eb_route_call;

typedef struct eb_route {
    int32_t kernel;        /* EB_ROUTE_* */
    int32_t chunk_bytes;   /* bytes of a row one lane loads at a time (0: plain kernel) */
    int32_t lanes, chunks; /* lanes per row, chunks per lane (team and wave kernel) */
    int32_t small_batch;   /* team kernel: small-batch mapping */
    int32_t narrow;        /* team kernel: one lane group per bag */
    int32_t non_temporal;  /* row loads bypass the caches */
    int32_t xcd_runs;      /* each XCD takes a contiguous run of workgroups */
    int32_t split;         /* wave kernel: waves per bag */
} eb_route;

/* Fills *route; returns 0. */
int eb_gather_route(const eb_route_call *call, eb_route *route);

#ifdef __cplusplus
}
#endif

#endif /* EB_ROUTE_H */
