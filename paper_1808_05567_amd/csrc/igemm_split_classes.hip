// The split kernel for the residue classes of a strided backward pass in one launch.
#include "igemm_split.h"

namespace convmi {

typedef void (*classes_fn_t)(const IgemmSplitClasses);
#define CLASSES_ENTRY(WK, WM, FM, KW, G, NI) {{WK, WM, FM, KW, G, NI, 1}, igemm_split_classes_kernel<WK, WM, FM, KW, G, NI>}
#define CLASSES_ENTRIES(WK, WM, FM, KW) \
    CLASSES_ENTRY(WK, WM, FM, KW, 1, 1), CLASSES_ENTRY(WK, WM, FM, KW, 1, 2), CLASSES_ENTRY(WK, WM, FM, KW, 1, 3)
static const struct ClassesEntry {
    IgemmSplitVariant v;
    classes_fn_t fn;
} g_classes[] = {
    CLASSES_ENTRIES(4, 1, 4, 1), CLASSES_ENTRIES(4, 1, 2, 1), CLASSES_ENTRIES(2, 2, 2, 1), CLASSES_ENTRIES(4, 1, 4, 2),
    CLASSES_ENTRIES(4, 1, 2, 2), CLASSES_ENTRIES(2, 2, 2, 2),
};

static const ClassesEntry *find(const IgemmSplitVariant &v)
{
    for (const ClassesEntry &e : g_classes)
        if (e.v.wk == v.wk && e.v.wm == v.wm && e.v.fm == v.fm && e.v.kw == v.kw && e.v.g == v.g && e.v.ni == v.ni) return &e;
    return nullptr;
}
bool igemm_split_classes_exist(const IgemmSplitVariant &v) { return find(v) != nullptr; }

hipError_t launch_igemm_split_classes(const IgemmSplitVariant &v, const IgemmSplitClasses &c, size_t lds_bytes, hipStream_t stream)
{
    const ClassesEntry *e = find(v);
    if (!e) return hipErrorInvalidDeviceFunction;
    if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(e->fn), lds_bytes); err != hipSuccess) return err;
    hipLaunchKernelGGL(e->fn, dim3(c.end[3]), dim3(256 * v.kw), lds_bytes, stream, c);
    return hipGetLastError();
}

}  // namespace convmi
