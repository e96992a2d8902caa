/* The index arithmetic of csrc/lgf_device.hpp as the host compiles it, for
 * ctypes. */
#include "lgf_device.hpp"

extern "C" {

// the quotients of n values by d
void probe_div(const uint32_t *values, uint32_t *quotients, int n, uint32_t d)
{
    const lgf::FastDiv f = lgf::make_fast_div(d);
    for (int i = 0; i < n; ++i) quotients[i] = lgf::fast_div(values[i], f);
}

// the place of every workgroup of a grid of n
void probe_places(uint32_t *places, uint32_t n, int order)
{
    for (uint32_t b = 0; b < n; ++b) places[b] = lgf::launch_place(b, n, order);
}

// the grid for n items over a lattice with t-slices of hs sites per parity; the
// first `room` workgroups' items
uint32_t probe_items(uint32_t *items, uint32_t room, uint32_t n, uint32_t Lt, uint32_t hs, uint64_t site_bytes)
{
    lgf::Geom g{};
    g.L[0] = Lt;
    g.hs[0] = hs;
    uint32_t grid = 0;
    const lgf::XcdRuns runs = lgf::xcd_runs(n, g, site_bytes, &grid);
    for (uint32_t b = 0; b < grid && b < room; ++b) items[b] = lgf::xcd_item(b, runs);
    return grid;
}

}  // extern "C"
