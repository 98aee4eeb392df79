"""What memory scene loads take from one another, without a GPU (fake_hip.c)."""
from test_launch_plans import fake  # noqa: F401  (a fixture)
from test_out_of_memory import _run


def test_scenes_of_about_one_size_follow_each_other(fake):  # noqa: F811
    """Twenty meshes, each a little larger than the one before: their 1.9 % of growth cross one step of sizes at most."""
    _run(fake, """
r = bps.bps_create(max_batch=1)
v, t = large.vertices, large.indices
for k in range(20):
    n = int(len(t) * (1 - 0.001 * (20 - k)))
    h = bps.bps_load_scene(r, v, t[:n])
    bps.bps_unload_scene(r, h)
assert bps.bps_query(r, 0, 8) <= 2 and fake.fake_allocated(1) <= 2, (bps.bps_query(r, 0, 8), fake.fake_allocated(1))
print("done")
""")


def test_a_small_scene_leaves_the_large_image_alone(fake):  # noqa: F811
    _run(fake, """
r = bps.bps_create(max_batch=1)
fake.fake_hold(1)      # copies take their time: an image for each
load(r, large)
load(r, small)
fake.fake_hold(0)
assert fake.fake_live(1) == 2
fake.fake_hold(1)
load(r, small)
load(r, large)
assert fake.fake_live(1) == 2
fake.fake_hold(0)
print("done")
""")
