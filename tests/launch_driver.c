/* Drives the library's host side with a HIP runtime of its own: the few runtime functions the library calls are defined here
 * and take the place of the real ones, so several devices and refusals can be played without a GPU.  No kernel runs and no
 * pointer is followed.  Checked: every device that a kernel with a large dynamic LDS block is launched on has granted it
 * that block beforehand, once, and a refusal is reported and not kept. */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "rdk.h"

typedef struct { uint32_t x, y, z; } dim3;

enum { kGrants = 256 };
static int g_device, g_refuse;
static struct { const void *kernel; int device, count; } g_grant[kGrants];
static int g_grants, g_launches, g_ungranted, g_twice;
static struct { dim3 grid, block; size_t shmem; void *stream; } g_config;

static int *grant_of(const void *kernel)
{
    for (int i = 0; i < g_grants; ++i)
        if (g_grant[i].kernel == kernel && g_grant[i].device == g_device) return &g_grant[i].count;
    return NULL;
}

static void *g_binary;
void **__hipRegisterFatBinary(const void *data) { (void)data; return &g_binary; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterFunction(void **m, const void *f, char *a, const char *b, unsigned t, void *c, void *d, void *e, void *g, int *w)
{
    (void)m; (void)f; (void)a; (void)b; (void)t; (void)c; (void)d; (void)e; (void)g; (void)w;
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
int hipGetDevice(int *device) { *device = g_device; return 0; }
int hipDeviceGetAttribute(int *value, int attr, int device) { (void)attr; (void)device; *value = 160 * 1024; return 0; }
int hipFuncSetAttribute(const void *kernel, int attr, int value)
{
    (void)attr; (void)value;
    if (g_refuse) return 1;
    int *n = grant_of(kernel);
    if (!n && g_grants < kGrants) {
        g_grant[g_grants].kernel = kernel;
        g_grant[g_grants].device = g_device;
        g_grant[g_grants].count = 0;
        n = &g_grant[g_grants++].count;
    }
    if (n && ++*n > 1) ++g_twice;
    return 0;
}
int hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **args, size_t shmem, void *stream)
{
    (void)grid; (void)block; (void)args; (void)stream;
    ++g_launches;
    if (shmem > 0 && !grant_of(kernel)) ++g_ungranted;
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

static void *at(uintptr_t x) { return (void *)(x << 20); }   /* a device pointer that nobody follows */

static rdk_status_t fused(const rdk_kernel_t *k, rdk_linear_mode_t mode)
{
    rdk_verify_desc_t d;
    memset(&d, 0, sizeof d);
    d.B = 4; d.N = 4096; d.sample_draft = 1;
    return rdk_redistribute_verify(k, mode, &d, at(1), RDK_PROB_F32, 4096, at(2), RDK_PROB_F32, 1024, NULL, 0, (int32_t *)at(3),
                                   (uint8_t *)at(4), NULL, NULL, (int32_t *)at(5), NULL, NULL, at(6), (size_t)1 << 30, NULL);
}

static int failures;
static void expect(int ok, const char *what, int device, int mode)
{
    if (!ok) {
        ++failures;
        printf("device %d, mode %d: %s\n", device, mode, what);
    }
}

int main(void)
{
    rdk_kernel_desc_t kd;
    memset(&kd, 0, sizeof kd);
    kd.N = 4096; kd.n = 1024; kd.kept_ids = (const int32_t *)at(7); kd.format = RDK_SPARSE_TOPK;   /* k = 0: no neighbours */
    rdk_kernel_t *kernel = NULL;
    if (rdk_build_kernel(&kd, at(8), (size_t)1 << 30, at(9), (size_t)1 << 30, NULL, &kernel) != RDK_OK) return 2;
    for (int device = 0; device < 70; device += device < 2 ? 1 : 23)   /* 0, 1, 2, 25, 48 */
        for (int mode = 0; mode < 2; ++mode) {
            const rdk_linear_mode_t m = mode ? RDK_LINEAR_SPARSE : RDK_LINEAR_TAYLOR;
            g_device = device;
            if (device) {
                g_refuse = 1;
                const int launched = g_launches;
                expect(fused(kernel, m) == RDK_ERR_HIP, "a refused grant is not reported", device, mode);
                expect(g_launches == launched, "launched without the grant", device, mode);
                g_refuse = 0;
            }
            for (int rep = 0; rep < 2; ++rep) expect(fused(kernel, m) == RDK_OK, "the call fails", device, mode);
            expect(g_ungranted == 0, "launched where the block was not granted", device, mode);
            expect(g_twice == 0, "granted again", device, mode);
            g_ungranted = g_twice = 0;
        }
    if (g_launches == 0 || g_grants == 0) return 2;   /* the library has not called the functions above */
    printf("%d launches, %d grants, %d failures\n", g_launches, g_grants, failures);
    return failures != 0;
}
