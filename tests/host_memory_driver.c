/* The library's use of device memory against a device of this file's making:
 * the HIP calls it makes are defined here, memory is a number of bytes and
 * kernels do nothing.  Prints "ok". */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "../include/mcx.h"
#include "../include/mcx_nn.h"

enum { kOutOfMemory = 2 };
static size_t g_used, g_limit = (size_t)64 << 30;
static struct { void *p; size_t n; } g_block[4096];
static int g_blocks, g_capturing, g_mallocs;

int hipMalloc(void **p, size_t n) {
  ++g_mallocs;
  if (g_used + n > g_limit) return kOutOfMemory;
  for (int i = 0; i < 4096; ++i)
    if (!g_block[i].p) {
      *p = g_block[i].p = malloc(n); /* never touched */
      g_block[i].n = n;
      g_used += n;
      ++g_blocks;
      return *p ? 0 : kOutOfMemory;
    }
  return kOutOfMemory;
}
int hipFree(void *p) {
  for (int i = 0; p && i < 4096; ++i)
    if (g_block[i].p == p) {
      g_used -= g_block[i].n;
      g_block[i].p = NULL;
      --g_blocks;
      free(p);
    }
  return 0;
}
int hipMemGetInfo(size_t *f, size_t *t) {
  *f = g_limit - g_used;
  *t = g_limit;
  return 0;
}
int hipStreamIsCapturing(void *s, int *st) { (void)s; *st = g_capturing; return 0; }
int hipThreadExchangeStreamCaptureMode(int *m) { (void)m; return 0; }
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return e == kOutOfMemory ? "out of memory" : "error"; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = &g_used; return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
int hipEventCreate(void **e) { *e = &g_used; return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = &g_used; return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.f; return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)d; (void)s; (void)n; (void)k; return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *t) {
  (void)d; (void)s; (void)n; (void)k; (void)t;
  return 0;
}
int hipMemsetAsync(void *d, int v, size_t n, void *s) { (void)d; (void)v; (void)n; (void)s; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t m) {
  (void)f; (void)b; (void)m;
  *n = 1;
  return 0;
}
int hipLaunchKernel() { return 0; }

#define CHECK(c)                                                       \
  do {                                                                 \
    if (!(c)) {                                                        \
      printf("line %d: %s; %s\n", __LINE__, #c, mcx_last_error());     \
      return 1;                                                        \
    }                                                                  \
  } while (0)

static mcx_nn *network(void) {
  const int32_t ch[2] = {32, 64};
  mcx_nn *nn = NULL;
  return mcx_nn_create(ch, 2, 32, 32, 32, 0, &nn) == MCX_OK ? nn : NULL;
}

/* a single-layer call of 1024 channels: leaves about 60 MB of scratch idle */
static mcx_status layer(void) {
  static uint16_t x[8 * 1024];
  static float w[1], y[1];
  return mcx_nn_layer_forward(MCX_NN_CONV3, 2, 2, 2, 1024, 1024, x, w, NULL, NULL, 0, 1, y, NULL);
}

static mcx_ctx *context(void) {
  static uint8_t labels[64 * 64 * 64];
  const mcx_medium media[2] = {{0, 0, 1, 1}, {0.005f, 1.f, 0.01f, 1.37f}};
  memset(labels, 1, sizeof(labels));
  mcx_sim sim;
  memset(&sim, 0, sizeof(sim));
  sim.vol.nx = sim.vol.ny = sim.vol.nz = 64;
  sim.vol.voxel_mm = 1.f;
  sim.vol.nmedia = 2;
  sim.vol.labels = labels;
  sim.vol.media = media;
  sim.src.pos[0] = sim.src.pos[1] = 31.5f;
  sim.src.dir[2] = 1.f;
  sim.gates.dt_ns = 0.5f;
  sim.gates.ngates = 10;
  sim.n_outside = 1.f;
  mcx_options o;
  mcx_default_options(&o);
  mcx_ctx *c = NULL;
  return mcx_batch_create(&sim, 1, &o, &c) == MCX_OK ? c : NULL;
}

int main(void) {
  /* what a network and a context take, and what a layer call leaves idle */
  mcx_nn *nn = network();
  CHECK(nn);
  const size_t of_network = g_used;
  mcx_nn_destroy(nn);
  CHECK(g_used == 0);
  mcx_ctx *c = context();
  CHECK(c);
  const size_t of_context = g_used;
  mcx_destroy(c);
  CHECK(g_used == 0);
  CHECK(layer() == MCX_OK);
  const size_t idle = g_used;
  CHECK(g_blocks == 1 && idle > ((size_t)50 << 20) && idle <= ((size_t)256 << 20));

  /* where they fit only with the idle memory given back, they are made */
  g_limit = of_network + idle / 2;
  CHECK((nn = network()));
  CHECK(g_used == of_network);
  mcx_nn_destroy(nn);
  g_limit = (size_t)64 << 30;
  CHECK(layer() == MCX_OK && g_used == idle);
  g_limit = of_context + idle / 2;
  CHECK((c = context()));
  CHECK(g_used == of_context);
  mcx_destroy(c);
  CHECK(g_used == 0);

  /* images that share launches: none with the network or under capture, once
     for all with the first call over symmetries, none where there is no room */
  static float phi[32 * 32 * 32], out[32 * 32 * 32];
  g_limit = (size_t)64 << 30;
  CHECK((nn = network()));
  const int before = g_mallocs;
  g_capturing = 1;
  CHECK(mcx_nn_forward_sym(nn, phi, out, NULL, 8, NULL) == MCX_OK);
  CHECK(g_used == of_network && g_mallocs == before);
  g_capturing = 0;
  CHECK(mcx_nn_forward_sym(nn, phi, out, NULL, 2, NULL) == MCX_OK);
  CHECK(g_used > of_network && g_mallocs == before + 1);
  CHECK(mcx_nn_forward_sym(nn, phi, out, NULL, 8, NULL) == MCX_OK && g_mallocs == before + 1);
  mcx_nn_destroy(nn);
  CHECK(g_used == 0);
  CHECK((nn = network()));
  g_limit = of_network + ((size_t)32 << 20);
  CHECK(mcx_nn_forward_sym(nn, phi, out, NULL, 8, NULL) == MCX_OK && g_used == of_network);
  mcx_nn_destroy(nn);
  CHECK(g_used == 0 && g_blocks == 0);
  printf("ok\n");
  return 0;
}
