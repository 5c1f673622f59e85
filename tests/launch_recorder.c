/* Records what the library would launch, without a GPU: this program defines the HIP runtime entry
 * points that the library calls (its own definitions are found before the runtime's), loads the
 * library, makes the calls that standard input describes on made-up addresses, and prints every
 * kernel launch.  Nothing is executed or dereferenced.
 *
 * input, one call per line:
 *   forward|static|backward T d_model d_ff E capacity_factor dtype ffn n_groups dropout jitter ntlb flags bias
 * output per call:
 *   call <status> <workspace address> <workspace bytes>
 *   launch <mangled kernel name> gx gy gz bx by bz lds <first three arguments, 8 bytes each>
 *   done
 * Usage: launch_recorder <library>
 */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

#include "switchffn.h"

typedef struct { uint32_t x, y, z; } Dim3;

static struct { const void *stub; const char *name; } kernels[2048];
static int n_kernels;
static Dim3 next_grid, next_block;
static size_t next_lds;
static void *next_stream;

/* ---- the HIP runtime as the library sees it ---- */
void **__hipRegisterFatBinary(const void *data) { (void)data; static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterFunction(void **modules, const void *stub, char *name, const char *device_name, unsigned limit,
                           void *tid, void *bid, void *bdim, void *gdim, int *wsize) {
    (void)modules; (void)device_name; (void)limit; (void)tid; (void)bid; (void)bdim; (void)gdim; (void)wsize;
    if (n_kernels == 2048) abort();
    kernels[n_kernels].stub = stub;
    kernels[n_kernels++].name = strdup(name);
}
void __hipRegisterVar(void **modules, void *var, char *name, char *device_name, int ext, size_t size, int constant,
                      int global) {
    (void)modules; (void)var; (void)name; (void)device_name; (void)ext; (void)size; (void)constant; (void)global;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream) {
    next_grid = grid; next_block = block; next_lds = lds; next_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream) {
    *grid = next_grid; *block = next_block; *lds = next_lds; *stream = next_stream;
    return 0;
}
int hipLaunchKernel(const void *stub, Dim3 grid, Dim3 block, void **args, size_t lds, void *stream) {
    (void)stream;
    const char *name = "?";
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].stub == stub) name = kernels[i].name;
    printf("launch %s %u %u %u %u %u %u %zu", name, grid.x, grid.y, grid.z, block.x, block.y, block.z, lds);
    if (strstr(name, "router_split_kernel"))   /* (W_r, wsplit, wsplit_b, ...) */
        for (int i = 0; i < 3; ++i) printf(" %llu", (unsigned long long)*(uint64_t *)args[i]);
    printf("\n");
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipGetDevice(int *dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int *value, int attr, int dev) { (void)attr; (void)dev; *value = 256; return 0; }
int hipFuncSetAttribute(const void *stub, int attr, int value) { (void)stub; (void)attr; (void)value; return 0; }
int hipGetSymbolAddress(void **ptr, const void *symbol) { (void)symbol; *ptr = (void *)(1ull << 40); return 0; }

int main(int argc, char **argv) {
    void *lib = argc == 2 ? dlopen(argv[1], RTLD_NOW) : NULL;
    if (!lib) { fprintf(stderr, "%s\n", argc == 2 ? dlerror() : "usage: launch_recorder <library>"); return 2; }
    int (*size_of)(const switch_config *, size_t *) = dlsym(lib, "switch_workspace_size");
    typeof(&switch_forward) forward = dlsym(lib, "switch_forward");
    typeof(&switch_forward_static) forward_static = dlsym(lib, "switch_forward_static");
    typeof(&switch_backward) backward = dlsym(lib, "switch_backward");
    char what[16];
    long long T, d, f, E, n;
    double cf;
    int dtype, ffn, ntlb, flags, bias;
    float dropout, jitter;
    while (scanf("%15s %lld %lld %lld %lld %lf %d %d %lld %f %f %d %d %d", what, &T, &d, &f, &E, &cf, &dtype, &ffn, &n,
                 &dropout, &jitter, &ntlb, &flags, &bias) == 14) {
        switch_config c = {T, d, f, E, cf, 0.01f, dtype, ffn, n, dropout, jitter, 17, ntlb, flags};
        size_t bytes = 0;
        int st = size_of(&c, &bytes);
        /* far apart, aligned, never touched */
        void *at = (void *)(1ull << 44), *ws = (void *)(1ull << 45);
        float *opt = bias ? at : NULL;
        if (st == 0 && strcmp(what, "forward") == 0)
            st = forward(&c, at, at, opt, at, at, at, at, at, at, at, at, at, NULL, ws, bytes, NULL);
        else if (st == 0 && strcmp(what, "static") == 0)
            st = forward_static(&c, at, at, opt, at, at, at, at, at, at, at, at, at, NULL, NULL);
        else if (st == 0)
            st = backward(&c, at, 1.f, at, at, opt, at, at, at, at, opt, at, at, ws, bytes, NULL);
        printf("call %d %llu %zu\ndone\n", st, (unsigned long long)(uintptr_t)ws, bytes);
    }
    fflush(stdout);
    _exit(0);   /* no destructors: there is no runtime to shut down */
}
