"""What the profiler and eclip_model_tune launch, on a runtime that only writes down which kernels it is given."""
import pytest

import fake_runtime

pytestmark = pytest.mark.skipif(not fake_runtime.HAVE, reason="needs hipcc")

PROGRAM = """
import paper_2506_12598_amd as ec
import workloads as wl
import workloads.graphs as graphs
side, cin, hidden, n, batch, cus = {sizes}
b = graphs._Builder("bottleneck", wl.DT_BF16, 1, graphs.IN_IMAGE, 8, side, side)
x = b.conv(-1, cin, 1)
y = b.conv(x, hidden, 1, act=wl.ACT_RELU6)
d = b.conv(y, hidden, 3, 1, 1, wl.ACT_RELU6, groups=hidden)
z = b.conv(d, n, 1)
b.maxpool(z, 1, 1, 0)
m = b.finish()
pool = ec.Pool([(ec.eclip_mask_layout(256, 32, 2, 0, cus // 32), 0)])
h = ec.Model(pool, m, wl.to_storage(m.weights, m.dtype), batch)
print(h.{call})
"""
SMALL = (14, 32, 96, 24, 2, 256)


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    tmp = str(tmp_path_factory.mktemp("fake"))
    lib = fake_runtime.build(tmp)
    return lambda call, sizes=SMALL, **env: fake_runtime.run(lib, tmp, PROGRAM.format(call=call, sizes=sizes), **env)


@pytest.mark.parametrize("call", ["tune(0, batch=2, iters=1)", "profile_group(0, 0, 2, 1)", "profile_group_served(0, 0, 2, 1)"])
def test_layers_that_share_a_launch_are_written_before_they_are_timed(launches, call):
    # timed one by one, the pointwise layer reads what the depthwise layer left; in one launch with the expansion it leaves nothing
    _, kernels = launches(call, ECLIP_EXPDW="1")
    convs = [k for k in kernels if "conv" in k or "expdw" in k]
    depthwise = [i for i, k in enumerate(convs) if "dwconv" in k]
    assert depthwise and depthwise[0] <= 2, convs[:6]                 # behind the first convolution and the expansion
    assert ("served" in call) == any("expdw" in k for k in convs)


@pytest.mark.parametrize("env,timed", [({"ECLIP_EXPDW": "1"}, 2), ({}, 3), ({"ECLIP_EXPDW": "0"}, 3)])
def test_a_pointwise_layer_in_one_launch_with_its_expansion_is_not_tuned(launches, env, timed):
    # 56 x 56 pixels, 16 -> 144 -> 96 channels on 64 CUs: two of the layers do not share a launch, and three only when told to.  The first convolution and the
    # expansion have plans that requests may read, the last layer only where the three are apart.
    out, _ = launches("tune(0, batch=1, iters=1)", (56, 16, 144, 96, 1, 64), **env)
    assert int(out) == timed
