/*
 * Drives the C ABI over a HIP runtime that refuses memory on request
 * (tests/test_gpu_runtime.py): this program's own hipMalloc and
 * hipHostMalloc stand before the runtime's for the library too.
 *
 * runtime_main deep GAME
 *     solves a small game that its one-block form leaves to the general
 *     path, with no further memory to be had; prints "deep status n_major
 *     n_valuations" for a whole run and for one with max_major = 2.
 *
 * runtime_main pairs GAME
 *     a best response refused in its first valuation (the last but one
 *     vertex is Even and answers with the last), then one that is not;
 *     prints "pairs status bytes" twice, the bytes held on the device with
 *     the cache given back.
 *
 * runtime_main idle GAME
 *     a batch leaves its memory for the next one; prints "idle status" of a
 *     load that finds no other memory.
 * runtime_main exact
 *     an arena just past powers of two that are not to be had; prints
 *     "exact status".
 *
 * runtime_main stale GAME
 *     calls after another HIP call of the thread failed and left its error
 *     behind; prints "stale status" of a load and of a poll of two games.
 *
 * GAME (little endian): int64 n, int64 m, int64 offsets[n+1], int32
 * targets[m], uint8 owner[n], int32 pri[n].
 */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "../include/pg.h"

#define HIP_OUT_OF_MEMORY 2

int hipSetDevice(int device);

#define MOST_BLOCKS 65536

static int refuse;
static struct { void *p; size_t bytes; } blocks[MOST_BLOCKS];
static int n_blocks;
static size_t held, most = (size_t)-1;   /* device bytes */

int hipMalloc(void **p, size_t bytes)
{
    static int (*next)(void **, size_t);
    if (!next)
        next = (int (*)(void **, size_t))dlsym(RTLD_NEXT, "hipMalloc");
    if (refuse || n_blocks == MOST_BLOCKS || held + bytes > most)
        return HIP_OUT_OF_MEMORY;
    int rc = next(p, bytes);
    if (rc == 0) {
        blocks[n_blocks].p = *p;
        blocks[n_blocks++].bytes = bytes;
        held += bytes;
    }
    return rc;
}

int hipFree(void *p)
{
    static int (*next)(void *);
    if (!next) next = (int (*)(void *))dlsym(RTLD_NEXT, "hipFree");
    for (int i = 0; i < n_blocks; ++i)
        if (blocks[i].p == p) {
            held -= blocks[i].bytes;
            blocks[i] = blocks[--n_blocks];
            break;
        }
    return next(p);
}

int hipHostMalloc(void **p, size_t bytes, unsigned flags)
{
    static int (*next)(void **, size_t, unsigned);
    if (!next)
        next = (int (*)(void **, size_t, unsigned))dlsym(RTLD_NEXT,
                                                         "hipHostMalloc");
    return refuse ? HIP_OUT_OF_MEMORY : next(p, bytes, flags);
}

typedef struct {
    int64_t n, m, *off;
    int32_t *tgt, *pri;
    uint8_t *owner;
} game;

static void *part(FILE *f, size_t size, int64_t count)
{
    void *p = malloc(size * (size_t)count);
    if (!p || fread(p, size, (size_t)count, f) != (size_t)count) {
        fprintf(stderr, "short game file\n");
        exit(3);
    }
    return p;
}

static game read_game(const char *path)
{
    game g;
    FILE *f = fopen(path, "rb");
    if (!f || fread(&g.n, 8, 1, f) != 1 || fread(&g.m, 8, 1, f) != 1)
        exit(3);
    g.off = part(f, 8, g.n + 1);
    g.tgt = part(f, 4, g.m);
    g.owner = part(f, 1, g.n);
    g.pri = part(f, 4, g.n);
    fclose(f);
    return g;
}

static pg_status load(const game *g, pg_game **out)
{
    return pg_load_csr(g->n, g->m, g->off, g->tgt, g->owner, g->pri, 0, NULL,
                       out);
}

static int deep(const char *path)
{
    game g = read_game(path);
    uint8_t *winner = malloc((size_t)g.n);
    for (int cap = 0; cap <= 2; cap += 2) {
        pg_game *d = NULL;
        pg_solve_opts o;
        pg_stats st;
        memset(&o, 0, sizeof o);
        o.max_major = cap;
        if (load(&g, &d) != PG_OK) return 2;
        refuse = 1;
        pg_status rc = pg_solve(d, &o, winner, NULL, NULL, &st, NULL);
        refuse = 0;
        printf("deep %d %lld %lld\n", (int)rc, (long long)st.n_major,
               (long long)st.n_valuations);
        pg_free(d);
        pg_release_cache();
    }
    return 0;
}

static int pairs(const char *path)
{
    game g = read_game(path);
    pg_game *d = NULL;
    int64_t na = 0;
    if (load(&g, &d) != PG_OK || pg_game_info(d, 0, 0, &na, 0) != PG_OK)
        return 2;
    int32_t *sigma = malloc(4 * (size_t)na), *tau = malloc(4 * (size_t)na);
    if (pg_initial_strategies(d, sigma, tau, 0, NULL) != PG_OK) return 2;
    for (int k = 0; k < 2; ++k) {
        sigma[g.n - 2] = k ? PG_SINK : (int32_t)(g.n - 1);
        pg_status rc = pg_best_response(d, sigma, tau, NULL, NULL, 0, 0,
                                        NULL);
        pg_release_cache();
        printf("pairs %d %lld\n", (int)rc, (long long)held);
    }
    return 0;
}

static int idle(const char *path)
{
    game g = read_game(path);
    pg_game *d = NULL;
    pg_batch *b = NULL;
    if (pg_batch_create(1 << 20, 8 << 20, 16, NULL, &b) != PG_OK) return 2;
    pg_batch_free(b);
    most = held;
    printf("idle %d\n", (int)load(&g, &d));
    return 0;
}

static int exact(void)
{
    const int64_t v = (1 << 21) + 1, e = (1 << 23) + 1;
    pg_batch *b = NULL;
    if (pg_batch_create(v, e, 16, NULL, &b) != PG_OK) return 2;
    const size_t all = held;
    pg_batch_free(b);
    pg_release_cache();
    most = held + (all - held) / 4 * 3;
    printf("exact %d\n", (int)pg_batch_create(v, e, 16, NULL, &b));
    return 0;
}

static int stale(const char *path)
{
    game g = read_game(path);
    pg_game *d = NULL;
    pg_batch *b = NULL;
    int64_t t[2];
    int32_t done[2] = {0, 0};
    uint8_t *w[2];
    if (pg_batch_create(1 << 18, 1 << 20, 16, NULL, &b) != PG_OK) return 2;
    for (int k = 0; k < 2; ++k)
        if (pg_batch_submit(b, g.n, g.m, g.off, g.tgt, g.owner, g.pri, 0,
                            &t[k]) != PG_OK ||
            hipHostMalloc((void **)&w[k], (size_t)g.n, 0) != 0)
            return 2;
    for (int32_t live = 1, queued = 1; live + queued > 0;)
        if (pg_batch_step(b, &live, &queued, NULL) != PG_OK) return 2;
    if (hipSetDevice(1000) == 0) return 2;
    printf("stale %d\n", (int)load(&g, &d));
    if (hipSetDevice(1000) == 0) return 2;
    printf("stale %d\n", (int)pg_batch_poll_many(b, 2, t, done, w, NULL, NULL,
                                                 NULL, 0));
    return !(done[0] && done[1]);
}

int main(int argc, char **argv)
{
    if (argc == 3 && !strcmp(argv[1], "deep")) return deep(argv[2]);
    if (argc == 3 && !strcmp(argv[1], "pairs")) return pairs(argv[2]);
    if (argc == 3 && !strcmp(argv[1], "idle")) return idle(argv[2]);
    if (argc == 2 && !strcmp(argv[1], "exact")) return exact();
    if (argc == 3 && !strcmp(argv[1], "stale")) return stale(argv[2]);
    fprintf(stderr, "usage: runtime_main MODE [GAME]\n");
    return 64;
}
