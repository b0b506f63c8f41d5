/*
 * Runs calls of the C ABI without a GPU and prints what they launch.  The program defines the few
 * HIP entry points that a launch goes through, so the library calls these instead of the
 * runtime's: kernels are logged by name with their grid and never run, and a launch can be made
 * to fail.  Device pointers are made up and never dereferenced.
 *
 * Reads one command a line from stdin:
 *   ctx T_max D F n_ffn n_zero n_copy n_const k act     a new context
 *   variant V | fail 0/1/2 (2: the next launch only) | capacity C (-1: off) | balance TAU
 *   forward T k | route T k | permute T k | ffn T k | combine T k
 * and prints "launch NAME gx gy gz threads" per kernel and "status S" per command.
 */
#define _GNU_SOURCE
#include "moepp.h"

#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim;

static struct { const void *host; char name[512]; } table[1024];
static int n_table, fail_launch, last_error;

void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned limit,
                           void *tid, void *bid, dim *block, dim *grid, int *wsize)
{
    typedef void (*fn)(void **, const void *, char *, const char *, unsigned, void *, void *, dim *, dim *, int *);
    fn real = (fn)dlsym(RTLD_NEXT, "__hipRegisterFunction");
    if (n_table < 1024) {
        table[n_table].host = host;
        snprintf(table[n_table++].name, sizeof table[0].name, "%s", name);
    }
    real(modules, host, device, name, limit, tid, bid, block, grid, wsize);
}

static dim cfg_grid, cfg_block;
static size_t cfg_shared;
static void *cfg_stream;
int __hipPushCallConfiguration(dim grid, dim block, size_t shared, void *stream)
{
    cfg_grid = grid;
    cfg_block = block;
    cfg_shared = shared;
    cfg_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim *grid, dim *block, size_t *shared, void **stream)
{
    *grid = cfg_grid;
    *block = cfg_block;
    *shared = cfg_shared;
    *stream = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void *host, dim grid, dim block, void **args, size_t shared, void *stream)
{
    (void)args;
    (void)shared;
    (void)stream;
    if (fail_launch) {
        if (fail_launch == 2) fail_launch = 0;
        return last_error = 719;
    }
    last_error = 0;                                 /* only the last call's error is kept */
    const char *name = "?";
    for (int i = 0; i < n_table; ++i)
        if (table[i].host == host) name = table[i].name;
    printf("launch %s %u %u %u %u\n", name, grid.x, grid.y, grid.z, block.x * block.y * block.z);
    return 0;
}
int hipGetLastError(void)
{
    const int e = last_error;
    last_error = 0;
    return e;
}
int hipGetDevice(int *dev) { return *dev = 0; }
int hipDeviceGetAttribute(int *value, int attribute, int dev)
{
    (void)attribute;
    (void)dev;
    *value = 256;                                   /* the only attribute the library asks for: CUs */
    return 0;
}

int main(void)
{
    char line[256], cmd[32];
    moepp_ctx *c = NULL;
    moepp_desc d;
    memset(&d, 0, sizeof d);
    void *p = (void *)0x100000;
    float *f = (float *)p;
    while (fgets(line, sizeof line, stdin)) {
        double v[9] = {0};
        if (sscanf(line, "%31s %lf %lf %lf %lf %lf %lf %lf %lf %lf", cmd, v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6,
                   v + 7, v + 8) < 1)
            continue;
        const int T = (int)v[0], k = (int)v[1];
        int st = -100;
        if (!strcmp(cmd, "ctx")) {
            const moepp_desc n = {T, k, (int)v[2], (int)v[3], (int)v[4], (int)v[5], (int)v[6], (int)v[7], (int)v[8]};
            if (c) moepp_destroy(c);
            c = NULL;
            d = n;
            st = moepp_create(&d, p, (size_t)1 << 60, &c);
        } else if (!strcmp(cmd, "variant")) {
            st = moepp_set_variant(c, T);
        } else if (!strcmp(cmd, "fail")) {
            fail_launch = T;
            st = 0;
        } else if (!strcmp(cmd, "capacity")) {
            int32_t cap[64];
            for (int i = 0; i < 64; ++i) cap[i] = T;
            st = moepp_set_capacity(c, T < 0 ? NULL : cap);
        } else if (!strcmp(cmd, "balance")) {
            st = moepp_set_balance(c, v[0]);
        } else if (!strcmp(cmd, "forward")) {
            st = moepp_layer_forward(c, NULL, T, p, f, f, f, p, p, f, k, p, f);
        } else if (!strcmp(cmd, "route")) {
            st = moepp_route(c, NULL, T, p, f, f, f, f, k, f);
        } else if (!strcmp(cmd, "permute")) {
            st = moepp_permute(c, NULL, T, k);
        } else if (!strcmp(cmd, "ffn")) {
            st = moepp_expert_ffn(c, NULL, T, p, p, k);
        } else if (!strcmp(cmd, "combine")) {
            st = moepp_combine(c, NULL, T, p, p, k, p);
        }
        printf("status %d\n", st);
    }
    if (c) moepp_destroy(c);
    return 0;
}
