"""Flags of the compilation units (CPU)."""
from paper_2106_12631_amd import build


def test_rambo_of_the_gradient_is_built_alike_everywhere():
    # RAMBO runs in rambo_grad.hip, and in the generated gradient units where
    # the gradient overwrites an input: with other flags its sums contract to
    # other multiply-adds and f depends on whether the call is in place
    for flag in build.source_flags('generated/grad_ggttg.hip'):
        assert flag in build.source_flags('rambo_grad.hip')
