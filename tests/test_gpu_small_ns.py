"""Newton-Schulz of small matrices by grouped launches: tile edges on both
sides, one row, one column, wide and tall; more shape groups than one launch
takes; and steps that mix the grouped items with tiled and Gram-space ones of
the same pool (equal padded short side)."""
import pytest
import torch

from oracle import normpre_oracle as O
from paper_2609_36692_amd import normpre as N
from paper_2609_36692_amd import workloads as WL
from parity_util import check_update

pytestmark = pytest.mark.gpu

# fp16 Newton-Schulz operands through five iterations.
TOL = 2e-2

SETS = {
    "one": [(1, 1)],
    "edges": [(64, 63), (65, 64), (1, 300), (300, 1), (255, 256), (257, 256), (129, 511)],
    # ten groups: two launches per stage
    "ten": [(40 + 60 * i, 500 - 45 * i) for i in range(10)],
    # (300, 330) grouped; the others take tiles, (256, 2048) in Gram space
    "mixed": [(300, 330)] + [(256, 2048)] * 10 + [(200, 256)] + [(250, 256)] * 50 + [(1024, 1500)] * 3,
}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = N.normpre_init(0)
    yield c
    N.normpre_destroy(c)


@pytest.mark.parametrize("variant", ["G", "MUON"])
@pytest.mark.parametrize("t", [0, 1])
@pytest.mark.parametrize("name", list(SETS))
def test_small_ns(ctx, name, t, variant):
    print(f"small Newton-Schulz {name} {variant} t={t}", flush=True)
    shapes = SETS[name]
    wl = WL.Workload("t", 90, shapes, "lowrank", 1.0, rank=8)
    mats = [WL.make_matrix(wl, i, "cpu", shape=s) for i, s in enumerate(shapes)]
    Ws, Gs, Ms = ([m[i].cuda().clone() for m in mats] for i in range(3))
    hp = N.normpre_default_hparams(lr=1.0, weight_decay=0.0, step=t)
    N.normpre_step(ctx, N.VARIANTS[variant], Ws, Gs, Ms, hp)
    torch.cuda.synchronize()
    ohp = O.HParams(lr=1.0, weight_decay=0.0)
    for i in sorted({shapes.index(s) for s in shapes} | {len(shapes) - 1}):
        w, g, m = (x.numpy() for x in mats[i])
        ref = (O.muon_step(w, g, m, ohp) if variant == "MUON"
               else O.normpre_step(w, g, m, t, ohp, variant, matrix_id=i))
        check_update(f"{variant} small {shapes[i]} t={t}",
                     mats[i][0].double().numpy() - Ws[i].cpu().double().numpy(), ref["update"], TOL)


# A small item beside tiled ones of its pool shares their launches; only the
# combines of Gram-space (two) and of tall items (one per iteration) are launched
# per item.  A chain of its own would be 15 launches.
@pytest.mark.parametrize("small,tiled,own", [((512, 512), [(512, 700)] * 8, 0), ((512, 2048), [(512, 4096)] * 24, 2),
                                             ((700, 500), [(700, 512)] * 8, 5)])
def test_small_item_stays_with_its_pool(ctx, small, tiled, own):
    classes = (N.NORMPRE_KCLASS_NS_GRAM, N.NORMPRE_KCLASS_NS_POLY, N.NORMPRE_KCLASS_NS_COMBINE)
    hp = N.normpre_default_hparams(step=0, flags=N.NORMPRE_FLAG_TIME_KERNELS)
    count = []
    for shapes in (tiled, [small] + tiled):
        Ws, Gs, Ms = ([torch.randn(s, device="cuda") for s in shapes] for _ in range(3))
        for c in classes:
            N.normpre_kernel_stats(ctx, c, reset=True)
        N.normpre_step(ctx, N.NORMPRE_VARIANT_G, Ws, Gs, Ms, hp)
        count.append(sum(N.normpre_kernel_stats(ctx, c)["launches"] for c in classes))
    print(f"Newton-Schulz launches {small} beside {tiled[0]}: {count}", flush=True)
    assert count[1] - count[0] <= own


# The grouped launches compute what the tiled ones do, bit by bit (the Muon
# step has no sum of its output): a matrix alone, and beside large ones of its
# pool, with which it takes the tiled launches.
@pytest.mark.parametrize("shape", [(100, 300), (129, 300), (300, 330), (512, 2048), (2048, 300), (768, 2000)])
def test_grouped_equals_tiled(ctx, shape):
    print(f"grouped against tiled {shape}", flush=True)
    wl = WL.Workload("t", 91, [shape], "lowrank", 1.0, rank=8)
    mat = [x.cuda() for x in WL.make_matrix(wl, 0, "cpu", shape=shape)]
    s = (min(shape) + 255) // 256 * 256
    out = []
    for beside in ([], [(s, 16384)] * 6):
        Ws, Gs, Ms = ([x.clone()] + [torch.randn(b, device="cuda") for b in beside] for x in mat)
        N.normpre_step(ctx, N.NORMPRE_VARIANT_MUON, Ws, Gs, Ms, N.normpre_default_hparams(lr=1.0, weight_decay=0.0))
        out.append(Ws[0].cpu())
    assert torch.equal(out[0], out[1])
