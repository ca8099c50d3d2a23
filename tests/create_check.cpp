// ds_create and ds_destroy against a stand-in for the HIP runtime, without a GPU: the functions below
// take the place of the runtime's (an executable's symbols come first), device memory is host
// memory, and a clear is carried out when something waits for the default stream, as late as the
// runtime may do it.  Called by test_create_cpu.py; exit status 0 and one line per check.
#include "../include/ds.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

namespace {
struct Clear {
    void *at;
    int value;
    size_t bytes;
};
std::vector<Clear> pending;
int allocations, clears, copies, live;

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
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *v, const void *, int, size_t) { *v = 4; return 0; }
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
}  // namespace

int main()
{
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
