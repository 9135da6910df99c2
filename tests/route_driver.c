/* Which kernels a call of the library launches, and with which grids: the few HIP runtime functions the library calls are defined here
 * and note the launches.  No kernel runs and no pointer is followed, so no GPU is needed.  Reads one call per line and answers each
 * with one line: status, bytes of workspace, then "name gx gy gz threads" per launch, separated by semicolons.  Input kinds, modes
 * and formats are the numbers of rdk.h:
 *   kernel FORMAT N n k          what the calls below work with
 *   exact QKIND B
 *   linear MODE PKIND QKIND B
 *   fused MODE PKIND QKIND B KEEP
 *   draft QKIND B
 *   multi PKIND B N C BYTES      workspace of BYTES, or of what the library asks for if negative
 */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "rdk.h"

typedef struct { uint32_t x, y, z; } dim3;

enum { kKernels = 4096 };
static struct { const void *host; const char *name; } g_kernel[kKernels];
static int g_kernels;
static struct { dim3 grid, block; size_t shmem; void *stream; } g_config;
static int g_noting;

static void *g_binary;
void **__hipRegisterFatBinary(const void *data) { (void)data; return &g_binary; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterFunction(void **m, const void *f, char *a, const char *b, unsigned t, void *c, void *d, void *e, void *g, int *w)
{
    (void)m; (void)a; (void)t; (void)c; (void)d; (void)e; (void)g; (void)w;
    if (g_kernels < kKernels) {
        g_kernel[g_kernels].host = f;
        g_kernel[g_kernels++].name = b;
    }
}
void __hipRegisterVar(void **m, void *v, char *a, char *b, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)a; (void)b; (void)e; (void)s; (void)c; (void)g;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, void *stream)
{
    g_config.grid = grid; g_config.block = block; g_config.shmem = shmem; g_config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, void **stream)
{
    *grid = g_config.grid; *block = g_config.block; *shmem = g_config.shmem; *stream = g_config.stream;
    return 0;
}
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int *value, int attr, int device) { (void)attr; (void)device; *value = 160 * 1024; return 0; }
int hipFuncSetAttribute(const void *kernel, int attr, int value) { (void)kernel; (void)attr; (void)value; return 0; }
int hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **args, size_t shmem, void *stream)
{
    const char *name = "unknown";
    (void)args; (void)shmem; (void)stream;
    if (!g_noting) return 0;
    for (int i = 0; i < g_kernels; ++i)
        if (g_kernel[i].host == kernel) name = g_kernel[i].name;
    printf(";%s %u %u %u %u", name, grid.x, grid.y, grid.z, block.x * block.y * block.z);
    return 0;
}
int hipExtLaunchKernel(const void *k, dim3 g, dim3 b, void **a, size_t s, void *st, void *e0, void *e1, int f)
{
    (void)e0; (void)e1; (void)f;
    return hipLaunchKernel(k, g, b, a, s, st);
}
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return e ? "refused" : "no error"; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = (void *)0x10000; return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)d; (void)s; (void)n; (void)k; (void)st; return 0; }
int hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, int k, void *st)
{
    (void)d; (void)dp; (void)s; (void)sp; (void)w; (void)h; (void)k; (void)st;
    return 0;
}
int hipStreamSynchronize(void *st) { (void)st; return 0; }
int hipEventCreate(void **e) { *e = (void *)1; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0; return 0; }

static void *at(uintptr_t x) { return (void *)(x << 44); }   /* a device pointer that nobody follows */

int main(void)
{
    const size_t room = (size_t)1 << 43;
    rdk_kernel_t *kernel = NULL;
    int N = 0, n = 0;
    char line[256], what[16];
    while (fgets(line, sizeof line, stdin)) {
        long a[5] = {0, 0, 0, 0, 0};
        size_t bytes = 0;
        rdk_status_t rc = RDK_OK;
        if (sscanf(line, "%15s %ld %ld %ld %ld %ld", what, a, a + 1, a + 2, a + 3, a + 4) < 2) return 2;
        g_noting = strcmp(what, "kernel") != 0;
        if (!strcmp(what, "kernel")) {
            rdk_kernel_desc_t d;
            memset(&d, 0, sizeof d);
            d.format = (rdk_kernel_format_t)a[0];
            d.N = N = (int)a[1]; d.n = n = (int)a[2]; d.k = (int)a[3];
            d.d = 64; d.tau = 0.1f;
            d.kept_ids = (const int32_t *)at(1);
            if (d.format != RDK_IDENTITY) d.embeddings = (const float *)at(2);
            if (kernel) rdk_destroy_kernel(kernel);
            kernel = NULL;
            rc = rdk_build_kernel(&d, at(3), room, at(4), room, NULL, &kernel);
        } else if (!strcmp(what, "exact")) {
            rc = rdk_workspace_bytes(kernel, (int)a[1], &bytes);
            printf("%d %zu", rc, bytes);
            rc = rdk_redistribute_exact(kernel, at(5), (rdk_input_kind_t)a[0], n, (int)a[1], (float *)at(6), N, at(7), bytes, NULL);
        } else if (!strcmp(what, "linear")) {
            rc = rdk_workspace_bytes(kernel, (int)a[3], &bytes);
            printf("%d %zu", rc, bytes);
            rc = rdk_redistribute_linear(kernel, (rdk_linear_mode_t)a[0], at(8), (rdk_input_kind_t)a[1], N, at(5), (rdk_input_kind_t)a[2], n,
                                         (int)a[3], (float *)at(6), N, at(7), bytes, NULL);
        } else if (!strcmp(what, "fused")) {
            rdk_verify_desc_t d;
            memset(&d, 0, sizeof d);
            d.B = (int)a[3]; d.N = N; d.sample_draft = 1;
            rc = rdk_redistribute_verify_workspace_bytes(kernel, (rdk_linear_mode_t)a[0], &d, &bytes);
            printf("%d %zu", rc, bytes);
            rc = rdk_redistribute_verify(kernel, (rdk_linear_mode_t)a[0], &d, at(8), (rdk_input_kind_t)a[1], N, at(5),
                                         (rdk_input_kind_t)a[2], n, a[4] ? (float *)at(6) : NULL, N, (int32_t *)at(9), (uint8_t *)at(10),
                                         (float *)at(11), (float *)at(12), (int32_t *)at(13), NULL, NULL, at(7), bytes, NULL);
        } else if (!strcmp(what, "draft")) {
            rc = rdk_sample_draft_workspace_bytes(kernel, (int)a[1], &bytes);
            printf("%d %zu", rc, bytes);
            rc = rdk_sample_draft(kernel, at(5), (rdk_input_kind_t)a[0], n, (int)a[1], 1, 0, (int32_t *)at(9), NULL, NULL, 0, at(7), bytes, NULL);
        } else if (!strcmp(what, "multi")) {
            rdk_multi_desc_t d;
            memset(&d, 0, sizeof d);
            d.B = (int)a[1]; d.N = (int)a[2]; d.C = (int)a[3];
            rc = rdk_verify_multi_workspace_bytes(&d, (rdk_input_kind_t)a[0], &bytes);
            printf("%d %zu", rc, bytes);
            rc = rdk_verify_multi(&d, at(8), (rdk_input_kind_t)a[0], d.N, (const float *)at(6), d.N, (int32_t *)at(9), (int32_t *)at(10),
                                  (int32_t *)at(11), NULL, at(7), a[4] < 0 ? bytes : (size_t)a[4], NULL);
        } else {
            return 2;
        }
        if (!g_noting) printf("%d 0", rc);
        printf(";%d\n", rc);
    }
    return 0;
}
