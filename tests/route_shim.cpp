// C entry over csrc/attn_route.h for tests/test_route_cpu.py.
#include "../paper_2603_24517_amd/csrc/attn_route.h"

extern "C" int route(int B, int Hq, int Hkv, int Sq, int Skv, int causal, int ncu, long long *out)
{
    attn::Route r = {};
    const int rc = attn::make_shape(B, Hq, Hkv, Sq, Skv, r.shape, r.sched);
    if (rc != ATTN_OK) return rc;
    attn::make_route(B, Hkv, Skv, causal, ncu, r);
    out[0] = r.kind;
    out[1] = r.kind == attn::ROUTE_SPLIT ? (long long)r.split.nrest * r.split.ntile : r.sched.total;            // work items
    out[2] = r.kind == attn::ROUTE_SPLIT ? out[1] * r.split.splits
                                         : r.kind == attn::ROUTE_SHARED ? r.share.wgs : 8 * r.sched.slots;      // workgroups
    out[3] = r.kind == attn::ROUTE_SPLIT ? r.split.units : r.kind == attn::ROUTE_SHARED ? r.share.units : 0;    // pool units
    out[6] = r.rows.kgroups;
    out[4] = r.kind == attn::ROUTE_SPLIT && r.split.once;
    out[5] = r.kind == attn::ROUTE_SPLIT && (r.split.once || r.split.once_region);                              // on the null stream
    return ATTN_OK;
}

// The steps that are enqueued for a call if the runtime takes all but step `refused` (-1: all), as letters in `log`.
extern "C" int steps(int B, int Hq, int Hkv, int Sq, int Skv, int causal, int ncu, int refused, int region, char *log)
{
    attn::Route r = {};
    const int rc = attn::make_shape(B, Hq, Hkv, Sq, Skv, r.shape, r.sched);
    if (rc != ATTN_OK) return rc;
    attn::make_route(B, Hkv, Skv, causal, ncu, r);
    return attn::enqueue(r, [&](attn::Step s) { *log++ = "TMG"[s]; return s != refused; }, region != 0);
}

extern "C" long long pool_bytes() { return (long long)attn::POOL_UNITS * attn::POOL_UNIT_BYTES; }

extern "C" int pool_units() { return attn::POOL_UNITS; }
extern "C" int region_units() { return attn::REGION_UNITS; }
extern "C" int sets_counters_back(unsigned unit) { return attn::sets_counters_back(unit); }

extern "C" void split_limits(long long *out)
{
    out[0] = attn::SPLIT_MAX_ITEMS;
    out[1] = attn::SPLIT_MAX_WGS;
    out[2] = attn::SPLIT_MAX_UNITS;
    out[3] = (attn::SPLIT_HEADER_BYTES / 4) - 1;
}
