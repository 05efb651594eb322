"""Groups of bfloat16 products too large for the memory-side cache: their
aligned products run the grouped kernels' form for operands that come from
HBM.  Every single-stage program and the mixed one, ragged sizes from 1 up
among the large ones, accumulation, and the CASE choice; small-integer
operands, so that every sum is exact, with NaN in the rows' padding."""
import pytest
import torch

from paper_1801_04348_amd import pk

pytestmark = pytest.mark.gpu

TILES = [(64, 64), (128, 64), (64, 128), (128, 128)]
EDGES = [(1, 1, 1), (3, 8, 5), (65, 63, 7), (64, 64, 64), (70, 130, 65), (129, 72, 127), (200, 9, 129), (5, 300, 191),
         (128, 128, 0), (131, 257, 193)]


@pytest.fixture(scope="module")
def table():
    return pk.pk_case_table_build(0)


def product(M, N, K, gen, lead=0):
    """A, B (bfloat16 views of NaN-padded rows), their exact product's C."""
    def operand(r, c):
        buf = torch.full((r, -(-max(c, 1) // 8) * 8 + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
        view = buf[:, lead:lead + c]
        view.copy_(torch.randint(-8, 9, (r, c), generator=gen, device="cuda"))
        return view
    a, b = operand(M, K), operand(K, N)
    return a, b, a.float() @ b.float()


@pytest.fixture(scope="module")
def group():
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    dims = EDGES + [(256 + 8 * (i % 33), 300 - i % 71, 200 + 3 * (i % 91)) for i in range(260)]
    return [product(*d, gen) for d in dims]


def outputs(group, value):
    return [torch.full((r.shape[0], r.shape[1] + 3), value, device="cuda")[:, :r.shape[1]] for _, _, r in group]


def check(plan, group, Cs, base, names):
    assert sorted(set(n.split("_", 3)[3] for n in plan.kernels())) == names, plan.kernels()
    plan.run()
    torch.cuda.synchronize()
    for (a, b, ref), C in zip(group, Cs):
        assert torch.equal(C, ref + base), (a.shape, b.shape)


@pytest.mark.parametrize("bm,bn", TILES)
@pytest.mark.parametrize("accumulate", [False, True])
def test_uniform(table, group, bm, bn, accumulate):
    p = pk.params(family=pk.PK_FAMILY_MFMA, variant=pk.PK_MFMA_SINGLE, bm=bm, bn=bn, bk=64, wm=2, wn=2)
    Cs = outputs(group, 2.0 if accumulate else float("nan"))
    plan = pk.pk_grouped_plan_create(table, "bf16", [x[0] for x in group], [x[1] for x in group], Cs,
                                     params=[p] * len(group), accumulate=accumulate)
    name = "%dx%dx64_w2x2_st1" % (bm, bn)
    check(plan, group, Cs, 2.0 if accumulate else 0.0, [name + "_el", name + "_hb"])  # (_el: the product without a K)


def test_mixed(table, group):
    ps = [pk.params(family=pk.PK_FAMILY_MFMA, variant=pk.PK_MFMA_SINGLE, bm=bm, bn=bn, bk=64, wm=2, wn=2)
          for bm, bn in (TILES[g % 4] for g in range(len(group)))]
    Cs = outputs(group, float("nan"))
    plan = pk.pk_grouped_plan_create(table, "bf16", [x[0] for x in group], [x[1] for x in group], Cs, params=ps)
    check(plan, group, Cs, 0.0, ["bf16_w2x2_st1_el", "bf16_w2x2_st1_hb"])


def test_choice_by_the_groups_size(table, group):
    wide = [x for x in group if x[0].shape[1] > 0]
    for part, form in ((wide, "_hb"), (wide[:150], "")):
        Cs = outputs(part, float("nan"))
        plan = pk.pk_grouped_plan_create(table, "bf16", [x[0] for x in part], [x[1] for x in part], Cs)
        assert all(n.endswith("_hb") == (form == "_hb") for n in plan.kernels()), plan.kernels()
        plan.capture()
        for _ in range(3):
            for C in Cs:
                C.fill_(float("nan"))
            plan.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(C, x[2]) for C, x in zip(Cs, part))


def test_unaligned_products_among_them(table, group):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    mixed = group + [product(100, 90, 80, gen, lead=1) for _ in range(3)]
    Cs = outputs(mixed, float("nan"))
    plan = pk.pk_grouped_plan_create(table, "bf16", [x[0] for x in mixed], [x[1] for x in mixed], Cs)
    plan.run()
    torch.cuda.synchronize()
    assert any(n.endswith("_hb") for n in plan.kernels()) and any(n.endswith("_el") for n in plan.kernels())
    assert all(torch.equal(C, x[2]) for C, x in zip(Cs, mixed))
