// The library's host side against a stand-in for the HIP runtime, without a GPU: the functions below
// take the place of the runtime's (an executable's symbols come first), device memory is host
// memory, a clear is carried out when something waits for the default stream, as late as the
// runtime may do it, and a launch is written down instead of carried out.  Called by test_create_cpu.py:
//   create_check           ds_create and ds_destroy; one line per check, exit status 0 if all hold
//   create_check launches  reads "block comp n d dtype flags [k]" lines (block w: worker, s: server and update in one
//                          call, p: the same without momentum; k: top-k entries, else d / 100 + 1) and prints the launches of that call: name and grid, one line each, then a dot
#include "../include/ds.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Clear {
    void *at;
    int value;
    size_t bytes;
};
std::vector<Clear> pending;
int allocations, clears, copies, live;

struct Grid {
    unsigned x, y, z;
};
// functions by their address in the host program, filled in while the library is loaded
std::map<const void *, std::string> &kernels()
{
    static std::map<const void *, std::string> k;
    return k;
}

// Workgroups of 512 threads per compute unit: those that hold R tiles in registers and L in LDS are built for
// 64, 80 and 128 registers.
int resident(const void *f)
{
    const std::string &name = kernels()[f];
    const size_t at = name.find("_held"), end = name.find("EEEv", at == std::string::npos ? 0 : at);
    if (at == std::string::npos || end == std::string::npos) return 4;
    const size_t l = name.rfind("Li", end), r = name.rfind("Li", l - 1);
    const int in_registers = atoi(name.c_str() + r + 2);
    return in_registers <= 4 ? 4 : in_registers <= 8 ? 3 : 2;
}

void carry_out()
{
    for (const Clear &c : pending) memset(c.at, c.value, c.bytes);
    pending.clear();
}
}  // namespace

extern "C" {
int hipMalloc(void **p, size_t bytes)
{
    *p = malloc(bytes);
    if (!*p) return 2;
    memset(*p, 0xA5, bytes);                     // what the memory held before
    ++allocations;
    ++live;
    return 0;
}
int hipFree(void *p)
{
    carry_out();
    live -= p != nullptr;
    free(p);
    return 0;
}
int hipHostMalloc(void **p, size_t bytes, unsigned) { return hipMalloc(p, bytes); }
int hipHostFree(void *p) { return hipFree(p); }
int hipMemset(void *at, int value, size_t bytes) { ++clears; pending.push_back({at, value, bytes}); return 0; }
int hipMemcpy(void *dst, const void *src, size_t bytes, int) { ++copies; carry_out(); memcpy(dst, src, bytes); return 0; }
int hipStreamSynchronize(void *) { carry_out(); return 0; }
int hipDeviceSynchronize() { carry_out(); return 0; }
int hipGetLastError() { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *v, const void *f, int, size_t) { *v = resident(f); return 0; }

void **__hipRegisterFatBinary(const void *)
{
    static void *module;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    kernels()[f] = name;
}
int hipGetSymbolAddress(void **, const void *) { return 1; }
static Grid pushed[2];
int __hipPushCallConfiguration(Grid grid, Grid block, size_t, void *)
{
    pushed[0] = grid;
    pushed[1] = block;
    return 0;
}
int __hipPopCallConfiguration(Grid *grid, Grid *block, size_t *lds, void **stream)
{
    *grid = pushed[0];
    *block = pushed[1];
    *lds = 0;
    *stream = nullptr;
    return 0;
}
int hipLaunchKernel(const void *f, Grid grid, Grid, void **, size_t, void *)
{
    printf("%s %u %u\n", kernels()[f].c_str(), grid.x, grid.y);
    return 0;
}
}

namespace {
int bad;

void expect(bool ok, const char *what, const char *name)
{
    printf("%s: %s: %s\n", ok ? "ok" : "FAILED", name, what);
    bad += !ok;
}

ds_config_t config(int comp, int n, int64_t d, int flags = 0)
{
    ds_config_t c;
    memset(&c, 0, sizeof c);
    c.comp = comp; c.n = n; c.d = d; c.flags = flags;
    c.levels = 15; c.bucket = 512; c.k = d / 100 + 1; c.chunk = 2048;
    return c;
}

// every word that a kernel expects cleared is cleared before ds_create returns
void cleared_before_the_first_call(const char *name, const ds_config_t &cfg)
{
    ds_ctx_t *c = nullptr;
    const ds_status_t rc = ds_create(&cfg, &c);
    expect(rc == DS_OK, "is created", name);
    expect(pending.empty(), "no clear is left for after ds_create", name);
    ds_destroy(c);
    expect(live == 0, "everything is given back", name);
}
// what creating a context asks of the runtime: allocations, and transfers that the host waits for
void creation_cost(const char *name, const ds_config_t &cfg, int most_allocations, int most_transfers)
{
    allocations = clears = copies = 0;
    ds_ctx_t *c = nullptr;
    expect(ds_create(&cfg, &c) == DS_OK, "is created", name);
    expect(allocations <= most_allocations, "allocations", name);
    expect(clears + copies <= most_transfers, "clears and copies", name);
    ds_destroy(c);
}
int launches()
{
    char block;
    int comp, n, dtype, flags;
    long long d, k;
    char line[256];
    while (fgets(line, sizeof line, stdin)) {
        const int fields = sscanf(line, " %c %d %d %lld %d %d %lld", &block, &comp, &n, &d, &dtype, &flags, &k);
        if (fields < 6) return 1;
        ds_config_t cfg = config(comp, n, d, flags);
        if (fields == 7) cfg.k = k;
        cfg.grad_dtype = dtype;
        ds_ctx_t *c = nullptr;
        if (ds_create(&cfg, &c) != DS_OK) return 1;
        // never read or written: no launch is carried out
        alignas(16) static char any[16];
        ds_payload_t p;
        p.sign_words = reinterpret_cast<uint64_t *>(any);
        p.scales = reinterpret_cast<float *>(any);
        p.levels = reinterpret_cast<uint8_t *>(any);
        p.pairs = reinterpret_cast<ds_pair_t *>(any);
        p.dense = reinterpret_cast<float *>(any);
        float *f = reinterpret_cast<float *>(any);
        const ds_status_t rc = block == 'w' ? ds_worker_compress(c, 0, any, d, f, d, &p, nullptr)
                                            : ds_server_aggregate_compress_update(c, 0, &p, f, &p, f, block == 's' ? f : nullptr, 0.1f, 0.9f, nullptr);
        printf(rc == DS_OK ? ".\n" : "failed\n");
        ds_destroy(c);
    }
    return 0;
}

}  // namespace

int main(int argc, char **)
{
    if (argc > 1) return launches();
    const int nofb_sid = DS_FLAG_NO_ERROR_FEEDBACK | DS_FLAG_SERVER_IDENTITY;
    cleared_before_the_first_call("sign, one scale", config(DS_COMP_SIGN, 4, 300001));
    cleared_before_the_first_call("sign, one scale, deferred", config(DS_COMP_SIGN, 4, 300001, DS_FLAG_DEFERRED_ERROR));
    cleared_before_the_first_call("ternary", config(DS_COMP_TERNARY, 4, 300001, nofb_sid));
    cleared_before_the_first_call("top-k", config(DS_COMP_TOPK, 4, 300001));
    cleared_before_the_first_call("qsgd", config(DS_COMP_QSGD, 4, 300001));
    cleared_before_the_first_call("rsparse", config(DS_COMP_RSPARSE, 4, 300001));

    // before the 1-bit context with one scale held rows on chip it made 2 allocations and 6 copies, the ternary one
    // 5 allocations
    creation_cost("sign, one scale, one workgroup", config(DS_COMP_SIGN, 4, 1024), 3, 2);
    creation_cost("sign, one scale, many workgroups", config(DS_COMP_SIGN, 8, 11173962), 3, 2);
    creation_cost("sign, one scale, rows beyond the device", config(DS_COMP_SIGN, 2, 60000000), 1, 0);
    creation_cost("ternary", config(DS_COMP_TERNARY, 8, 11173962, nofb_sid), 6, 1);
    return bad ? 1 : 0;
}
