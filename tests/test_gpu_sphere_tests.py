"""The sphere-box tests spread over a wave's lanes, at the sizes where their
mapping changes: links with one sphere and with more than 32 (two chunks),
the most static boxes (32), objects with one and with 16 spheres, waves with
idle lanes (3, 5 and 6 steps), scenes far from the origin (the culling test's
margins), and batches in which most configurations are in contact.  Terms,
touching-pair counts and gradients against the FP64 oracle at the bars of
test_gpu_parity.py."""
import numpy as np
import pytest

import oracle as O
from paper_2411_11833_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _crowded(K, n_obstacles, seed):
    """Obstacles on a grid around the arm, so that most configurations touch
    several of them at once (make_scene keeps its boxes apart)."""
    rng = np.random.default_rng(seed)
    scene = I.make_scene(seed, n_objects=K, n_obstacles=0)
    xy = rng.uniform(-0.35, 0.35, (n_obstacles, 2))
    h = rng.uniform(0.05, 0.2, (n_obstacles, 3))
    scene.obstacles = np.concatenate([xy, rng.uniform(0.0, 0.6, (n_obstacles, 1)),
                                      rng.uniform(-3, 3, (n_obstacles, 1)), h], 1)
    return scene


def _robot(per_link):
    """The generated arm with `per_link[L]` spheres on link L + 1."""
    r = I.make_robot(0, n_spheres=60)
    rng = np.random.default_rng(1)
    sph, link = [], []
    for L, c in enumerate(per_link):
        base = r.spheres[r.sphere_link == L + 1]
        for _ in range(c):
            s = base[rng.integers(len(base))].copy()
            s[:3] += rng.uniform(-0.02, 0.02, 3)
            sph.append(s)
            link.append(L + 1)
    r.spheres, r.sphere_link = np.array(sph), np.array(link, dtype=np.int32)
    return r


def _case(name):
    if name == "link_of_70":
        p = I.Problem(_robot([1, 0, 1, 70, 3, 33, 0, 1]), _crowded(2, 6, 3), I.Skeleton(np.arange(2, dtype=np.int32)))
    elif name == "link_of_32":
        p = I.Problem(_robot([32, 1, 32, 31, 1, 2, 7, 5]), _crowded(4, 9, 4), I.Skeleton(np.arange(4, dtype=np.int32)))
    elif name == "boxes_32":
        p = I.Problem(I.make_robot(0, 60), _crowded(3, 31, 5), I.Skeleton(np.arange(3, dtype=np.int32)))
    elif name == "one_sphere_objects":
        sc = _crowded(5, 2, 6)
        sc.obj_spheres = sc.obj_spheres[:, :1] * np.array([0, 0, 0, 2.0])
        p = I.Problem(I.make_robot(0, 40), sc, I.Skeleton(np.arange(5, dtype=np.int32)))
    elif name == "objects_of_16":
        sc = _crowded(6, 4, 7)
        sc.obj_spheres = np.concatenate([sc.obj_spheres, sc.obj_spheres * np.array([0.5, 0.5, 0.5, 1.0])], 1)
        p = I.Problem(I.make_robot(0, 60), sc, I.Skeleton(np.arange(6, dtype=np.int32)))
    else:   # far boxes: only the culling sees them, and must not lose the near ones
        sc = _crowded(1, 12, 8)
        sc.obstacles[6:, :2] += np.array([[300.0, -700.0]])
        sc.obstacles[9:, 4:6] = 900.0   # a slab under everything, 700 m off centre
        sc.obstacles[9:, 2] = -0.05
        sc.obstacles[9:, 6] = 0.04
        sc.obstacles[9:, 3] = 0.0
        p = I.Problem(I.make_robot(0, 60), sc, I.Skeleton(np.arange(1, dtype=np.int32)))
    p.skeleton.goal_cost = int(p.skeleton.n_steps > 1)
    return p


@pytest.mark.parametrize("split", [1, 2, 4])
@pytest.mark.parametrize("name,n", [("link_of_70", 45), ("link_of_32", 77), ("boxes_32", 50),
                                    ("one_sphere_objects", 61), ("objects_of_16", 23), ("far", 131)])
def test_sphere_tests_match_oracle(name, n, split):
    from paper_2411_11833_amd.planner import GpuProblem
    prob = _case(name)
    gp = GpuProblem(prob)
    gp.set_split(split)
    X = I.uniform_particles(prob, n, seed=9)
    X64 = X.astype(np.float64)
    Xd = gp.from_rows(X)
    _, T, _ = gp.cost(Xd, n, terms=True)
    pairs = gp.penetrating_pairs(Xd, n)
    _, G = gp.cost_grad(Xd, n)
    torch.cuda.synchronize()
    To = O.terms(prob, X64)
    err = np.abs(gp.to_rows(T, n).cpu().numpy() - To)
    # far: positions stay near the origin, but the slab's FP32 box-frame offset
    # is 700 m, whose half ulp (3e-5 m) each touching sphere may be off by
    far = 6e-5 * 62 if name == "far" else 0.0
    assert np.all(err <= 1e-4 * np.abs(To) + 2e-6 + far), np.argwhere(err > 1e-4 * np.abs(To) + 2e-6 + far)[:5]
    want, close = O.penetrating_pairs(prob, X64, near=1e-6 if name != "far" else 1e-4)
    assert np.all(np.abs(pairs.cpu().numpy() - want) <= close)
    assert want.mean() > 5, "the batch is meant to be in contact"
    Jo, Go = O.cost_and_grad(prob, X64)
    _, kink = O.margins(prob, X64)
    ok = kink >= (1e-5 if name != "far" else 1e-4)
    d = np.linalg.norm(gp.to_rows(G, n).cpu().numpy() - Go, axis=1)
    bar = 1e-3 * np.linalg.norm(Go, axis=1) + 1e-5
    assert ok.any() and np.all(d[ok] <= bar[ok]), (np.flatnonzero(ok & (d > bar))[:5], d[ok & (d > bar)][:5])
