// Instantiations and dispatch of the split kernel (igemm_split.h).
#include "igemm_split.h"

namespace convmi {

#define SPLIT_FW false
static const SplitEntry g_split[] = {SPLIT_TABLE};

static const SplitEntry *find(const IgemmSplitVariant &v)
{
    int n = (int)(sizeof(g_split) / sizeof(g_split[0]));
    const SplitEntry *tab = v.fw ? igemm_split_fwd_wt_entries(&n) : g_split;
    for (int i = 0; i < n; ++i)
        if (tab[i].wk == v.wk && tab[i].wm == v.wm && tab[i].fm == v.fm && tab[i].kw == v.kw && tab[i].g == v.g && tab[i].ni == v.ni)
            return &tab[i];
    return nullptr;
}

bool igemm_split_exists(const IgemmSplitVariant &v) { return find(v) != nullptr; }

size_t igemm_split_lds_bytes(const IgemmSplitVariant &v, int pls)
{
    const size_t ring = (size_t)v.kw * 2 * 2 * v.g * pls * kPosBytes + (v.fw ? (size_t)v.kw * 4 * kWtBytes : 0);
    return std::max(ring, v.kw > 1 ? (size_t)4 * v.fm * 4096 : (size_t)0);
}

hipError_t launch_igemm_split(const IgemmSplitVariant &v, const IgemmArgs &a, size_t lds_bytes, int grid, hipStream_t stream)
{
    const SplitEntry *e = find(v);
    if (!e) return hipErrorInvalidDeviceFunction;
    if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(e->fn), lds_bytes); err != hipSuccess) return err;
    hipLaunchKernelGGL(e->fn, dim3(grid), dim3(256 * v.kw), lds_bytes, stream, a);
    return hipGetLastError();
}

}  // namespace convmi
