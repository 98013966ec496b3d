"""Options of the code generator that decide which branches stay branches: only the strict form, in which a region with a branch
that lanes may take differently, at any depth, is structurized as without the option; and only for the decode kernels, where it is
worth its while."""
from paper_2605_08317_amd import build


def test_regions_are_left_alone_only_where_every_branch_is_uniform():
    for source, obj, flags in build.SOURCES:
        skips = any("structurizecfg-skip-uniform-regions" in f for f in flags)
        strict = "-structurizecfg-relaxed-uniform-regions=false" in flags
        assert skips == strict, obj
        assert not skips or source.startswith("decode_m"), obj
    assert not any("structurizecfg" in f for f in build.FLAGS)
