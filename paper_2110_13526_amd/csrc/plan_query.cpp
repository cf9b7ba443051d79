// plan_query.cpp -- the kernel forms that a geometry takes, for tests of the rules that
// choose them (not part of kct.h; host arithmetic only, no device needed).
#include <string>
#include <vector>

#include "kct_forward.h"
#include "kct_internal.h"

namespace kct {

void set_error(const std::string &msg);
kct_status geometry_tables(const kct_volume_desc &vol, const kct_cone_desc &cone, std::vector<ColParam> &cols,
                           std::vector<RowParam> &rows, std::vector<ViewParam> &views, GeoDev &d);

}  // namespace kct

using namespace kct;

// out: forward rows per lane, divided, read in place, forward workgroups; backward form
// (BwdForm), brick depth, view subsets, bricks.
extern "C" kct_status kct_test_plan(const kct_volume_desc *vol, const kct_cone_desc *cone, int32_t projector,
                                    kct_dtype dtype, int64_t out[8])
{
    std::vector<ColParam> cols;
    std::vector<RowParam> rows;
    std::vector<ViewParam> views;
    GeoDev g{};
    const kct_status s = geometry_tables(*vol, *cone, cols, rows, views, g);
    if (s != KCT_OK) return s;
    g.projector = projector;
    const bool tt = projector == KCT_PROJECTOR_TT;
    const FwdPlan f = forward_plan(g);
    const BwdPlan b = tt ? tt_backward_plan(g) : backward_plan(g, dtype != KCT_F64);
    const int64_t v[8] = {f.rows, f.divided, forward_in_place(g), forward_num_blocks(g), b.form, b.tz, b.sets, b.nblocks};
    for (int i = 0; i < 8; ++i) out[i] = v[i];
    return KCT_OK;
}

// out: column group, view and row band of workgroup w of a forward projection with
// `rows` detector rows per lane; in_place: of one that reads the volume in its own layout.
extern "C" void kct_test_forward_tile(int32_t nu, int32_t nv, int32_t views, int32_t rows, int32_t in_place, int64_t w,
                                      int64_t out[3])
{
    GeoDev g{};
    g.nu = nu;
    g.nv = nv;
    g.nviews = views;
    int cg, k, band;
    if (in_place) fwd_tile_in_place(fwd_grid(g, rows), (unsigned)w, cg, k, band);
    else fwd_tile(fwd_grid(g, rows), (unsigned)w, cg, k, band);
    out[0] = cg;
    out[1] = k;
    out[2] = band;
}
