"""The planner (csrc/lbp_host.cpp, plain C++) compiled on its own and asked over random layers."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2309_15275_amd", "csrc")


def run(tmp_path, body):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src = tmp_path / "driver.cpp"
    src.write_text('#include "lbp_host.h"\n#include <algorithm>\n#include <cmath>\n#include <cstdio>\n#include <random>\nusing namespace lbp;\n'
                   "std::mt19937 rng(7);\n"
                   "long draw(double lo, double hi) { return std::lround(std::exp(std::uniform_real_distribution<double>(std::log(lo), std::log(hi))(rng))); }\n"
                   "size_t up(size_t v) { return (v + 255) / 256 * 256; }\n" + body)
    exe = tmp_path / "driver"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), os.path.join(CSRC, "lbp_host.cpp"), "-o", str(exe)],
                   check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stdout[-2000:])


def test_a_call_can_always_be_planned_into_what_its_plainest_form_needs(tmp_path):
    # projected tensors, one set of coefficients where the reverse projection is a kernel of its own, one fp32 weight
    # gradient: no plan of any version needs less, so a fixed workspace that took a call goes on taking it
    run(tmp_path, """
int main()
{
    for (int i = 0; i < 3000; ++i) {
        const int patches[] = {2, 4, 8, 8, 16};
        const int patch = patches[rng() % 5], dt = rng() % 2, m = dt == LBP_BF16 ? 8 : 4;
        lbp_shape_t s{(int)draw(1, 128), (int)draw(1, 56), (int)draw(1, 56), (int)(m * draw(1, 512)), (int)(m * draw(1, 512)), dt, LBP_F32};
        const int r = (int)draw(1, patch * patch), extra = rng() % 3;
        const long rows = patch_count(s.N, s.H, s.W, patch) * r + (long)s.N * extra;
        const size_t esz = dtype_size(dt), w4 = up((size_t)s.Cin * s.Cout * 4);
        const size_t proj = up(rows * s.Cout * esz) + up(rows * s.Cin * esz);
        WorkspacePlan ws, fast;
        for (int fuse = 0; fuse < 2; ++fuse) {
            size_t bound = proj + w4;
            if (dt == LBP_BF16) {
                const bool can = fuse && (patch == 4 || patch == 8), wide = rng() % 2 && patch == 8;
                const int coef16 = rng() % 2;
                if (!can) bound += up((size_t)rows * s.Cin * (coef16 && extra == 0 ? 2 : 4));
                plan_workspace(&s, patch, r, 256, can, false, &fast, wide, true, extra, coef16);
                plan_workspace(&s, patch, r, 256, can, false, &ws, wide, true, extra, coef16, 0, true);
            } else {
                if (!fuse || patch > 8) bound += up((size_t)rows * s.Cin * 4);
                plan_workspace_f32(&s, patch, r, fuse && patch <= 8, true, true, extra, &fast, 256);
                plan_workspace_f32(&s, patch, r, fuse && patch <= 8, true, true, extra, &ws, 256, 1);
            }
            if (ws.total > bound || ws.total > fast.total) {
                printf("%d %dx%d %d->%d dtype %d patch %d r %d extra %d fuse %d: %zu of %zu (fastest plan %zu)\\n", s.N, s.H, s.W, s.Cin, s.Cout, dt,
                       patch, r, extra, fuse, ws.total, bound, fast.total);
                return 1;
            }
        }
        plan_workspace(&s, 0, 0, 256, false, false, &ws, false, true, 0, 0, 0, true);
        if (dt == LBP_F32) plan_workspace_f32(&s, 0, 0, false, true, true, 0, &ws, 256, 1);
        if (ws.total > w4) return 2;
    }
    return 0;
}
""")


def test_tiles_and_slices_follow_the_number_of_compute_units(tmp_path):
    run(tmp_path, """
int main()
{
    // one unit runs the tiles one after the other: full ones, and nothing is cut into slices
    for (int t : {kTile128, kTile64})
        if (fused_tile_step(kGemmTiles[t], 640, 128, 256, 1, 8, 1) != kGemmTiles[t].bm || fused_tile_step(kGemmTiles[t], 640, 128, 256, 1, 8, 256) >= kGemmTiles[t].bm) return 1;
    if (f32_tile_step(640, 64, 256, 1, 8, 1) != 64 || f32_tile_step(640, 64, 256, 1, 8, 256) >= 64) return 2;
    for (int cus : {1, 64, 256}) {
        const F32Cut c = plan_f32_products(4, 8192, 12, 4096, cus);
        const int slices = 4 * c.splits_x + 12 * c.splits_w;
        printf("%d units: %d slices\\n", cus, slices);
        if (slices > std::max(16, 3 * cus + 16)) return 3;
    }
    return 0;
}
""")


def test_tiles_hold_few_patches_only_where_the_device_is_not_full(tmp_path):
    run(tmp_path, """
int patches(lbp_shape_t s, int r, int patch, int *most, int *join)
{
    WorkspacePlan ws;
    if (plan_workspace(&s, patch, r, 256, true, false, &ws, false, true) != LBP_OK || !ws.gx_fused || !ws.grouped || ws.gx_step % r) return -1;
    *most = kGemmTiles[ws.gx.tile].bm / r;
    *join = ws.gx_join;
    return ws.gx_step / r;
}
int main()
{
    int most, join;
    for (int r = 3; r <= 4; ++r)
        if (patches({64, 32, 32, 768, 3072, 1, 0}, r, 8, &most, &join) != most) return 10 + r;
    for (int r = 1; r <= 4; ++r)      // (r = 3: 294 tiles of 42 patches are one round of the device and a bit)
        if (patches({128, 32, 32, 768, 768, 1, 0}, r, 8, &most, &join) != most && r != 3) return 20 + r;
    if (patches({128, 32, 32, 768, 768, 1, 0}, 3, 8, &most, &join) >= most) return 23;
    if (patches({32, 16, 16, 1024, 4096, 1, 0}, 2, 8, &most, &join) != most || join < 2) return 30;
    if (patches({64, 16, 16, 768, 3072, 1, 0}, 2, 8, &most, &join) != most || join < 2) return 31;
    if (patches({42, 7, 7, 600, 1264, 1, 0}, 3, 8, &most, &join) >= most) return 40;      // little work
    if (patches({75, 13, 13, 160, 1712, 1, 0}, 2, 8, &most, &join) >= most) return 41;
    if (patches({54, 8, 8, 3096, 1400, 1, 0}, 2, 8, &most, &join) >= most) return 42;     // full, but with short workgroups of the other product
    if (patches({1, 26, 26, 1536, 2960, 1, 0}, 1, 8, &most, &join) >= most) return 43;
    if (patches({2, 7, 7, 3648, 2864, 1, 0}, 6, 8, &most, &join) >= most || join < 3) return 44;      // slices that would start late
    if (patches({3, 52, 52, 1816, 3560, 1, 0}, 4, 8, &most, &join) != most || join < 2) return 45;      // ... few of them and two slices: all instead
    return 0;
}
""")


def test_slices_are_planned_for_the_order_that_is_run(tmp_path):
    # launches of more workgroups than the device holds, cut into slices: whichever product the launch dispatches first, its planner must not
    # fall back on two launches for the sake of the other order (input gradient first, all patches, one launch: 0.70 to 1.005 of two)
    run(tmp_path, """
int main()
{
    int seen = 0;
    for (int i = 0; i < 60000; ++i) {
        lbp_shape_t s{(int)draw(1, 128), (int)draw(7, 56), (int)draw(7, 56), (int)(8 * draw(100, 512)), (int)(8 * draw(200, 512)), LBP_BF16, LBP_F32};
        const int r = (int)draw(1, 7);
        const long rows = patch_count(s.N, s.H, s.W, 8) * r;
        WorkspacePlan ws;
        plan_workspace(&s, 8, r, 256, true, false, &ws, false, true);
        if (!ws.grouped || ws.gx_join < 2 || ws.gx_step / r != kGemmTiles[ws.gx.tile].bm / r) continue;
        const long n = gemm_workgroups(ws.gx, rows, s.Cin, s.Cout, r, 8, 256, true) * ws.gx_join + gemm_workgroups(ws.gw, s.Cout, s.Cin, rows, 0, 0, 256);
        const long steps_x = ((s.Cout + ws.gx_join - 1) / ws.gx_join + 63) / 64, steps_w = ((rows + ws.gw.splits - 1) / ws.gw.splits + 63) / 64;
        // (where those slices have no room, two launches are asked for before one in one piece)
        if (ws.or_apart && (n <= 512 || weight_gradient_first(false, n, steps_x, steps_w, 256))) return 3;
        seen += ws.or_apart;
    }
    if (weight_gradient_first(false, 512, 1, 9, 256) || !weight_gradient_first(false, 513, 5, 5, 256) || !weight_gradient_first(false, 513, 6, 5, 256) ||
        weight_gradient_first(false, 513, 7, 5, 256) || weight_gradient_first(true, 513, 1, 9, 256)) return 2;
    printf("%d\\n", seen);
    return seen > 50 ? 0 : 1;
}
""")


def test_a_grouped_launch_cuts_the_weight_gradient_as_often_as_the_product_alone(tmp_path):
    # a slice is one chain of fp32 sums: fewer of them, whatever else the launch holds, would be further from the exact sums
    run(tmp_path, """
int main()
{
    int grouped = 0, cut = 0;
    for (int i = 0; i < 20000; ++i) {
        lbp_shape_t s{(int)draw(1, 170), (int)draw(7, 56), (int)draw(7, 56), (int)(8 * draw(9, 400)), (int)(8 * draw(1, 400)), LBP_BF16, LBP_F32};
        const int r = (int)draw(1, 40), patch = rng() % 4 ? 8 : 4;
        if (r > patch * patch) continue;
        const long rows = patch_count(s.N, s.H, s.W, patch) * r;
        WorkspacePlan ws;
        plan_workspace(&s, patch, r, 256, true, false, &ws, patch == 8 && r > 8, true, 0, 1);
        if (!ws.grouped || ws.gw.tile != kTile128) continue;
        const GemmPlan own = plan_gemm(s.Cout, s.Cin, rows, 4, true, 0, 0, 256, false, kTile128);
        if (ws.gw.splits < own.splits) {
            printf("%d %dx%d %d->%d r %d patch %d: %d slices of %d\\n", s.N, s.H, s.W, s.Cin, s.Cout, r, patch, ws.gw.splits, own.splits);
            return 1;
        }
        ++grouped;
        cut += own.splits > 2;
    }
    return grouped > 100 && cut > 100 ? 0 : 2;
}
""")


def test_bias_sums_beside_the_products_take_the_place_of_the_projected_input(tmp_path):
    # a call with a bias gradient brings its projected input along, so that place is free: no memory is added where the rows fit there
    run(tmp_path, """
int main()
{
    int there = 0, behind = 0;
    for (int i = 0; i < 5000; ++i) {
        const int patch = rng() % 4 ? 8 : 4;
        lbp_shape_t s{(int)draw(1, 128), (int)draw(7, 56), (int)draw(7, 56), (int)(8 * draw(6, 512)), (int)(8 * draw(6, 512)), LBP_BF16, LBP_BF16};
        const int r = (int)draw(1, 16), extra = rng() % 2;
        WorkspacePlan ws;
        plan_workspace(&s, patch, r, 256, true, false, &ws, false, true, extra);
        const size_t bytes = (size_t)patch_count(s.N, s.H, s.W, patch) * s.Cout * 4, at = bias_sums_beside(ws, bytes);
        if (at % 256 || at < ws.gy_r + (size_t)patch_count(s.N, s.H, s.W, patch) * r * s.Cout * 2) return 1;       // (not on g^y)
        if (at < ws.total) {
            if (at != ws.x_r || at + bytes > std::min(ws.gx_r, std::min(ws.splitk, ws.total))) return 2;     // (not on what products write)
            ++there;
        } else ++behind;
        if (r * s.Cin >= 2 * s.Cout && at >= ws.total) return 3;
    }
    return there > 500 && behind > 500 ? 0 : 4;
}
""")


# bytes of the largest plan without a bias gradient; rows of patch sums fit on the projected input
@pytest.mark.parametrize("layer, r, most", [((64, 14, 14, 768, 3072), 8, 75497472), ((64, 16, 16, 768, 3072), 8, 75497472),
                                            ((128, 56, 56, 96, 384), 8, 76431360), ((128, 32, 32, 768, 768), 16, 419168256)])
def test_reported_workspaces_do_not_grow_for_a_bias_gradient_that_has_its_place(layer, r, most):
    from paper_2309_15275_amd import binding
    n, h, w, cin, cout = layer
    assert 4 * cout <= 2 * r * cin
    assert binding.workspace_bytes(binding.LbpShape(n, h, w, cin, cout, 1, 0), 8, r) <= most


def test_a_network_of_many_layers_plans_each_of_them_once(tmp_path):
    # calls that come round, 300 distinct ones, cost about what four of them do: each is found among the kept plans (0.1 us, where planning anew
    # takes 2 to 20)
    run(tmp_path, """
#include <chrono>
double us_a_call(int layers, int rounds)
{
    const auto t0 = std::chrono::steady_clock::now();
    for (int k = 0; k < rounds; ++k)
        for (int i = 0; i < layers; ++i) {
            lbp_shape_t s{1 + i % 50, 16, 16, 768, 3072 + 8 * (i / 50), i % 2, LBP_F32};
            WorkspacePlan ws;
            if (i % 2 == LBP_F32) plan_workspace_f32(&s, 8, 8, true, true, true, 0, &ws, 256);
            else plan_workspace(&s, 8, 8, 256, true, false, &ws, false, true);
        }
    return std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / layers / rounds;
}
int main()
{
    double few = 1e300, many = 1e300;
    us_a_call(300, 2);
    for (int k = 0; k < 10; ++k) {
        few = std::min(few, us_a_call(4, 2000));
        many = std::min(many, us_a_call(300, 30));
    }
    printf("%.3f %.3f us\\n", few, many);
    return many < 10 * few + 0.2 ? 0 : 1;
}
""")


def test_workspaces_have_counters_of_their_own(tmp_path):
    # calls on different workspaces may overlap in time: no two may be given the same arrival counters, and none may change hands
    run(tmp_path, """
int main()
{
    CounterSets c;
    char ws[40];
    if (c.of(nullptr) != 0) return 1;
    for (int round = 0; round < 2; ++round)
        for (int i = 0; i < 40; ++i)
            if (c.of(ws + i) != (i < CounterSets::kSets - 1 ? i + 1 : -1)) return 2;
    return c.of(nullptr) == 0 ? 0 : 3;
}
""")


def _reads(tmp_path, cases, field, gx_follows=True):
    rows = ",\n".join("{%d, %d, %d, %d, %d, %d, %d, %d, %d}" % (H, W, patch, *words, *blocks, *want) for H, W, patch, words, blocks, want in cases)
    run(tmp_path, """
const long cases[][9] = {%s};
int main()
{
    int bad = 0;
    for (const auto &c : cases) {
        const ProjectionReads how = plan_projection_reads(c[0], c[1], c[2], c[3], c[5] * 256, c[4], c[6] * 256, %s);
        if (how.%s[0] == c[7] && how.%s[1] == c[8]) continue;
        printf("%%ld x %%ld patch %%ld words %%ld %%ld workgroups %%ld %%ld\\n", c[0], c[1], c[2], c[3], c[4], c[5], c[6]);
        bad = 1;
    }
    return bad;
}
""" % (rows, "true" if gx_follows else "false", field, field))


def test_runs_of_projection_workgroups_where_they_gain(tmp_path):
    # (H, W, patch, words and workgroups of either tensor, runs): rows of whole 128-byte lines alone and in pairs, whole and hanging patches;
    # other rows by how full the patches are and, less than half, by how their workgroups meet the units; launches of 2047 and 2048 workgroups
    _reads(tmp_path, [
        (14, 14, 8, (1536, 0), (1536, 0), (0, 0)), (14, 14, 8, (384, 0), (384, 0), (0, 0)), (14, 14, 8, (1536, 384), (1536, 384), (1, 1)),
        (16, 16, 8, (1536, 0), (1536, 0), (1, 0)), (14, 14, 8, (1536, 0), (2047, 0), (0, 0)), (14, 14, 8, (1536, 0), (2048, 0), (1, 0)),
        (14, 16, 4, (32, 0), (512, 0), (0, 0)), (9, 9, 8, (1052, 84), (1332, 107), (0, 1)), (9, 9, 8, (1052, 84), (1946, 107), (1, 1)),
        (9, 9, 8, (1052, 96), (1332, 102), (0, 1)), (9, 9, 8, (420, 0), (610, 0), (1, 0)), (9, 9, 8, (500, 0), (726, 0), (0, 0)),
        (11, 11, 8, (500, 0), (700, 0), (0, 0)), (11, 12, 8, (500, 0), (700, 0), (1, 0)), (5, 5, 4, (500, 0), (700, 0), (0, 0)), (7, 8, 8, (500, 0), (700, 0), (1, 0))], "runs")


def test_narrow_rows_are_read_through_the_caches_where_that_gains(tmp_path):
    # (..., cached): both narrow; one beside whole lines and beside wide rows, at the least workgroups; rows of 256 words are whole lines, 260 wide;
    # one tensor alone; 96 MiB of either (1536 workgroups of 8 x 8 patches) and more, where no input gradient follows
    _reads(tmp_path, [(16, 16, *c) for c in [
        (8, (24, 36), (3, 2), (1, 1)), (8, (24, 96), (64, 192), (1, 0)), (8, (24, 96), (63, 193), (0, 0)), (8, (24, 96), (64, 191), (0, 0)),
        (8, (300, 252), (400, 64), (0, 1)), (8, (300, 252), (400, 63), (0, 0)), (4, (300, 252), (400, 32), (0, 1)), (4, (300, 252), (400, 31), (0, 0)),
        (8, (256, 252), (400, 400), (0, 1)), (8, (260, 252), (400, 400), (0, 1)), (8, (252, 0), (400, 0), (0, 0)), (8, (24, 36), (1536, 1536), (1, 1)),
        (8, (24, 36), (1537, 1536), (0, 1)), (8, (24, 36), (1536, 1537), (0, 0)), (4, (24, 36), (6144, 6144), (1, 1)), (4, (24, 36), (6144, 6145), (0, 0))]],
           "cached", False)


def test_large_narrow_rows_in_front_of_an_input_gradient_keep_the_hint(tmp_path):
    # a workgroup of 8 x 8 patches is 65536 bytes, of which 49/64 are inside a 7 x 7 grid: both narrow up to 24 MB of x (366 workgroups; 478), x alone
    # up to 48 MB (732), gy alone up to 64 MB of itself (976) and 80 MB of x (1220)
    _reads(tmp_path, [(16, 16, 8, *c) for c in [
        ((24, 36), (300, 366), (1, 1)), ((24, 36), (300, 367), (0, 0)), ((24, 36), (976, 366), (1, 1)), ((24, 36), (977, 366), (0, 1)), ((300, 36), (300, 732), (0, 1)),
        ((300, 36), (300, 733), (0, 0)), ((64, 36), (3000, 732), (0, 1)), ((24, 300), (976, 1220), (1, 0)), ((24, 300), (977, 1220), (0, 0)), ((24, 300), (976, 1221), (0, 0))]] +
        [(7, 7, 8, (24, 36), (300, 478), (1, 1)), (7, 7, 8, (24, 36), (300, 479), (0, 0)), (16, 16, 4, (24, 36), (2000, 1464), (1, 1)), (16, 16, 4, (24, 36), (2000, 1465), (0, 0))], "cached")


def test_exact_gradients_on_tall_tiles(tmp_path):
    # 256 x 128 for products whose columns (an input gradient's) or rows (a weight gradient's) leave half of 128 x 256 tiles empty, and for input
    # gradients behind a weight gradient, one workgroup a unit; not with short reductions, not for the second alone
    from test_gpu_tall_tiles import CASES
    no = [(33000, 128, 512, "gx", ""), (5184, 936, 3648, "gx", ""), (5184, 936, 1536, "both", ""), (20000, 936, 3648, "both", "")]
    rows = ", ".join("{%d, %d, %d, %d, %d, %d}" % (m, cin, cout, grads == "both", tall == "gx", tall == "gW") for m, cin, cout, grads, tall in CASES + no)
    run(tmp_path, """
const int cases[][6] = {%s};
int main()
{
    for (const auto &c : cases) {
        lbp_shape_t s{1, 1, c[0], c[1], c[2], LBP_BF16, LBP_F32};
        WorkspacePlan ws;
        plan_workspace(&s, 0, 0, 256, false, false, &ws, false, c[3]);
        if ((c[4] && ws.gx.tile != kTileTall) || (c[5] && ws.gw.tile != kTileTall) || (!c[4] && !c[5] && ws.gx.tile == kTileTall)) {
            printf("%%d rows %%d -> %%d: %%d %%d\\n", c[0], c[1], c[2], ws.gx.tile, ws.gw.tile);
            return 1;
        }
    }
    return 0;
}
""" % rows)


def test_input_gradients_on_wide_tiles_where_they_gain():
    # one round of half as many workgroups, many rounds of lines; not where the last columns are mostly empty, with few steps, with more stores than
    # steps, or beside a weight gradient whose workgroups take much longer
    from paper_2309_15275_amd import binding
    from test_gpu_wide_tiles import BESIDE, LONE

    def wide(N, H, W, extra, cin, cout, patch, r, both):
        plan = binding.describe_plan(binding.LbpShape(N, H, W, cin, cout, 1, 0), patch, binding.select_bases(patch, r), extra=extra, want_gw=both, num_cus=256)
        return "gx: tile 128x256" in plan

    assert all(wide(*c, both=True) for c in BESIDE) and all(wide(*c, both=False) for c in LONE)
    assert not wide(10, 27, 27, 0, 3160, 744, 8, 18, both=True)          # 64 -> 73 us on wide tiles
    for c in [(55, 50, 53, 1, 576, 384, 8, 6), (15, 28, 28, 0, 752, 408, 8, 54), (31, 51, 51, 0, 1432, 1456, 8, 4), (107, 14, 14, 1, 552, 576, 4, 9)]:
        assert not wide(*c, both=False), c                               # 68 -> 73, 33 -> 35, 166 -> 174, 39 -> 44


def test_runs_of_matrix_core_projections(tmp_path):
    # whole lines never; others but for patches at most 9/16 full in fewer than 2048 workgroups
    run(tmp_path, """
int main()
{
    auto f = matrix_projection_runs;
    return !f(16, 16, 8, 128, 4096) && f(16, 16, 8, 136, 512) && f(13, 13, 8, 136, 600) && !f(12, 12, 8, 136, 600) && !f(9, 9, 8, 136, 2047) &&
                   f(9, 9, 8, 136, 2048) && !f(5, 5, 4, 72, 700) && f(5, 8, 4, 72, 700) ? 0 : 1;
}
""")
