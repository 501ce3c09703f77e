"""The audit of the step table (validate_steps) on planners with a mistake in them: what a step's kernel has no room for is refused
before anything is launched."""
import pytest

from tests import host_stub


def _refused(tmp_path, planted, net, **kw):
    path = host_stub.build(str(tmp_path / "planted.so"), planted)
    host_stub.run(path, f"""
net = {net!r}
try:
    engine(net, **{kw!r})
except B.PBError as e:
    assert 'bounds audit' in str(e), e
else:
    raise AssertionError('accepted')
""")


def _norm(c, g, hw):
    import pb_workloads as W
    st = [[W.conv(3, c, 1, 1, 0)], [W.gn(g, c), W.relu(), W.conv(c, 4, 1, 1, 0)], [W.gn(1, 4), W.relu(), W.gap(), W.linear(4, 5), W.ce()]]
    return W._net("norm", st, 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)


# more channels than the workgroup has sums for, more elements than its shares
@pytest.mark.parametrize("net", [_norm(2050, 2, 1), _norm(40, 1, 33)], ids=["channels", "elements"])
def test_walked_groups_beyond_their_limits_are_refused(tmp_path, net):
    _refused(tmp_path, {"if (n > GNB_STREAM_N || cpg > GNB_STREAM_CPG) return false;": "", "if (g_tile_budget_us <= 0) return n <= 5120;": "return true;"},
             net, tuning=dict(tile_budget_us=-1.0))


def test_projection_weights_at_the_end_of_the_arena_are_refused(tmp_path):
    """Vectors at the end of a row of no multiple of 4 weights reach up to 3 floats past them."""
    import pb_workloads as W
    st = [[W.conv(3, 5, 3, 1, 1)], [W.relu(), W.conv(5, 7, 3, 1, 1)], [W.relu(), W.conv(7, 7, 3, 1, 1), W.add(1, 5, 7, 1, 1)],
          [W.gn(1, 7), W.relu(), W.gap(), W.linear(7, 5), W.ce()]]
    plant = "const StepDesc& d = pr.second;\n    if (d.pmask) {"
    moved = ("StepDesc d = pr.second;\n    if (d.kind == K_GEMM && (d.flags & F_PROJ) && d.g.gm == 1)\n"
             "      d.wp = hi - (int64_t)(d.pdepth - 1) * d.pstride - (int64_t)d.K * d.sC;\n    if (d.pmask) {")
    _refused(tmp_path, {plant: moved}, W._net("projection", st, 3, 5, 5, 5, 1e-3, 0.9, 8, 3, 8))
