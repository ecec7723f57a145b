/* Stands in for the HIP runtime under libwise.so: a program linked with this
 * file records each kernel launch instead of running it.  It refuses what HIP
 * refuses, a grid of 2^32 threads or more in one dimension, and leaves the
 * error for hipGetLastError as HIP does.  Reads one call a line from stdin
 * (entry batch heads kv_heads seq_len head_dim block option) and prints the
 * launches and the status.  Pointers are never followed: host code only. */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "wise.h"

typedef struct { uint32_t x, y, z; } dim3_t;
typedef int hip_error;

static struct { const void* stub; char name[192]; } table[512];
static int entries;
static dim3_t grid_, block_;
static size_t lds_;
static hip_error last;
static void* handle;

void** __hipRegisterFatBinary(const void* data) { (void)data; return &handle; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) {
  (void)m, (void)v, (void)h, (void)d, (void)e, (void)s, (void)c, (void)g;
}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned n, void* a, void* b, void* c,
                           void* d, int* w) {
  (void)m, (void)dev, (void)n, (void)a, (void)b, (void)c, (void)d, (void)w;
  table[entries].stub = host;
  strncpy(table[entries++].name, name, sizeof table[0].name - 1);
}
hip_error __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* st) {
  (void)st;
  grid_ = g, block_ = b, lds_ = lds;
  return 0;
}
hip_error __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** st) {
  *g = grid_, *b = block_, *lds = lds_, *st = 0;
  return 0;
}
hip_error hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t lds, void* st) {
  (void)args, (void)st;
  const char* name = "?";
  for (int i = 0; i < entries; ++i)
    if (table[i].stub == f) name = table[i].name;
  const int ok = g.x > 0 && g.y > 0 && g.z > 0 && (uint64_t)g.x * b.x < (1ull << 32) && (uint64_t)g.y * b.y < (1ull << 32) &&
                 g.y < 65536 && g.z < 65536 && (uint64_t)b.x * b.y * b.z <= 1024 && lds <= 65536;
  printf("%s %s %u %u %u %u %zu\n", ok ? "launch" : "refused", name, g.x, g.y, g.z, b.x, lds);
  if (!ok) last = 9;
  return ok ? 0 : 9;
}
hip_error hipGetLastError(void) {
  const hip_error e = last;
  last = 0;
  return e;
}
hip_error hipGetDevice(int* d) { *d = 0; return 0; }
hip_error hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)4096; return 0; }

int main(void) {
  char entry[32];
  wise_shape s;
  int opt;
  void* p = (void*)4096;
  while (scanf("%31s %d %d %d %d %d %d %d", entry, &s.batch, &s.heads, &s.kv_heads, &s.seq_len, &s.head_dim, &s.block, &opt) == 8) {
    s.scale = 0.f;
    wise_status st = WISE_ERR_RANGE;
    int32_t* order = opt ? p : 0;
    if (!strcmp(entry, "dense")) st = wise_dense_attn_accum(&s, p, p, p, p, p, 0, 0, 0, 0);
    else if (!strcmp(entry, "mass")) st = wise_dense_attn_accum(&s, p, p, p, p, p, p, p, SIZE_MAX, 0);
    else if (!strcmp(entry, "select")) st = wise_select_support(&s, p, 0.9f, 3u, p, p, order, p, SIZE_MAX, 0);
    else if (!strcmp(entry, "noalloc")) st = wise_select_support_noalloc(&s, p, 0.9f, 3u, p, p, order, 0);
    else if (!strcmp(entry, "step")) st = wise_select_step(&s, p, 0.9f, p, 0);
    else if (!strcmp(entry, "masks")) st = wise_support_from_masks(&s, p, 2, 3u, p, p, order, p, SIZE_MAX, 0);
    else if (!strcmp(entry, "sparse")) st = wise_sparse_attn(&s, p, p, p, p, p, order, p, p, 0);
    else if (!strcmp(entry, "grouped")) st = wise_sparse_attn_grouped(&s, p, p, p, p, p, p, p, 0);
    else if (!strcmp(entry, "support")) st = wise_support_mass(&s, p, p, p, p, opt ? p : 0, 0);
    printf("status %d\n", (int)st);
  }
  return 0;
}
