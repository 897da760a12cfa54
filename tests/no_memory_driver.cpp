// Driver of test_no_memory_host.py: wcsim_plane_create on a host without a GPU
// while the library's allocations fail from the k-th on.  Every call has to
// return a status; an exception that reaches this caller fails the run.
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <new>
#include <vector>

#include "wcsim.h"

static long g_left = -1;  // allocations of the library still granted (-1: all)
static long g_live;       // its allocations not yet freed

static bool from_library(void *caller)
{
    Dl_info info;
    return dladdr(caller, &info) && info.dli_fname && strstr(info.dli_fname, "libwcsim");
}

static void *allocate(size_t n, void *caller)
{
    if (g_left >= 0 && from_library(caller)) {
        if (g_left == 0)
            return nullptr;
        --g_left;
    }
    return malloc(n ? n : 1);
}

void *operator new(size_t n)
{
    void *p = allocate(n, __builtin_return_address(0));
    if (!p)
        throw std::bad_alloc();
    ++g_live;
    return p;
}
void *operator new(size_t n, const std::nothrow_t &) noexcept
{
    void *p = allocate(n, __builtin_return_address(0));
    g_live += p != nullptr;
    return p;
}
void operator delete(void *p) noexcept
{
    g_live -= p != nullptr;
    free(p);
}
void operator delete(void *p, size_t) noexcept { operator delete(p); }

int main()
{
    std::vector<float> resp(21 * 20, 0.01f), elec(5, 1.0f);
    wcsim_plane_desc d;
    memset(&d, 0, sizeof d);
    d.nwires = 10;
    d.nimpact = 10;
    d.nticks = 100;
    d.pitch = 5.0;
    d.tick = 0.5;
    d.dir_z = 1.0;
    d.resp_npitch = 21;
    d.resp_nticks = 20;
    d.resp_origin = 10;
    d.response = resp.data();
    d.elec_nticks = 5;
    d.elec_response = elec.data();
    wcsim_physics ph;
    memset(&ph, 0, sizeof ph);
    ph.drift_speed = 1.6;
    ph.nsigma = 3.0;
    wcsim_schedule sc;
    memset(&sc, 0, sizeof sc);
    int bad = 0, none = 0;
    wcsim_plane *first = nullptr;  // (the runtime's own start, the message's buffer)
    if (wcsim_plane_create(&d, &ph, nullptr, &first) == WCSIM_OK)
        wcsim_plane_destroy(first);
    for (int k = 0; k < 40; ++k)
        for (int form = 0; form < 2; ++form) {
            wcsim_plane *pl = (wcsim_plane *)&d;  // (any value: the call clears it)
            const long live = g_live;
            wcsim_status st = WCSIM_OK;
            g_left = k;
            try {
                st = form ? wcsim_plane_create_with_schedule(&d, &ph, &sc, nullptr, &pl)
                          : wcsim_plane_create(&d, &ph, nullptr, &pl);
            } catch (...) {
                printf("allocation %d, form %d: an exception crossed the call\n", k, form);
                ++bad;
            }
            g_left = -1;
            none += st == WCSIM_E_NOMEM;
            // (no GPU: with memory enough the first device call fails)
            if (st == WCSIM_OK || pl || g_live > live + 2) {  // (the pool table's slot, the message)
                printf("allocation %d, form %d: status %d, plane %p, %ld live\n", k, form, (int)st,
                       (void *)pl, g_live - live);
                ++bad;
            }
        }
    printf("%d calls without memory %s\n", none, bad || none < 4 ? "FAILED" : "ok");
    return bad || none < 4;
}
