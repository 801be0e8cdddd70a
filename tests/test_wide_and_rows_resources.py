"""Generated code of the kernels with pairs of tiles and for few query rows: instances, and what a sweep waits for."""
import re

from tests.test_kernel_resources import _kernels, _waits_at_sweep_start, code_objects  # noqa: F401


def test_next_pair_does_not_wait_for_the_stores_before_it(code_objects):  # noqa: F811
    """Q and the first tiles of a pair are requested before the results of the pair ahead of it are stored, and its sweep waits for
    all but those stores: fewer would undo the overlap, and with more in flight the tiles would not have arrived.  The same for the
    single tiles behind the pairs."""
    kernels = {}
    for obj in code_objects:
        kernels.update(_kernels(obj, "attn_fwd_wide_kernel"))
    assert len(kernels) == 6                    # d = 128 and 64; fp32, bf16 results, base 2
    for name, code in kernels.items():
        d, bf16 = re.search(r"attn_fwd_wide_kernelILi(\d+)ELb\dELb(\d)E", name).groups()
        tile = (2 if bf16 == "1" else 4) * int(d) // 32 + 1          # stores of 32 rows: 64 bytes of 16 rows each, and the lse
        for stores in (2 * tile, tile):                              # of a pair's wavefront (64 rows), of a single tile's
            starts = _waits_at_sweep_start(code, stores)
            assert starts
            for waits in starts:
                if 0 in waits:      # in front of the loop, for the first item; behind such a wait inside the loop the compiler would add none for Q
                    waits = waits[len(waits) - waits[::-1].index(0):]
                    assert max(waits) > stores, (name, stores, starts)
                assert min(waits) >= stores, (name, stores, starts)


def test_stores_of_a_pair_follow_the_loads_it_waits_for(code_objects):  # noqa: F811
    """The count in that wait is the number of stores behind the loads: as many stand between the normalisation and the next
    sweep, none of them conditional."""
    for obj in code_objects:
        for name, code in _kernels(obj, "attn_fwd_wide_kernel").items():
            d, bf16 = re.search(r"attn_fwd_wide_kernelILi(\d+)ELb\dELb(\d)E", name).groups()
            wanted = 2 * ((2 if bf16 == "1" else 4) * int(d) // 32 + 1)
            runs, n = [], 0
            for op, _ in code:
                if op.startswith("buffer_store"):
                    n += 1
                elif op.startswith(("s_cbranch", "s_branch", "s_barrier")):
                    runs, n = runs + ([n] if n else []), 0
            assert wanted in runs, (name, wanted, runs)


def test_instances_for_few_rows(code_objects):  # noqa: F811
    kernels = {}
    for obj in code_objects:
        kernels.update(_kernels(obj, "attn_rows_kernel"))
    assert sorted(re.search(r"ILi(\d+)ELi(\d)ELi(\d)E", n).groups() for n in kernels) == [("128", "8", "1"), ("128", "8", "2"), ("64", "8", "1"), ("64", "8", "2")]
