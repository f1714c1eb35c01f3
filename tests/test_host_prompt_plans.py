"""Which prompt GEMMs the cases of test_gpu_prompt_plans.py launch (host code over a recorded HIP runtime, no GPU)."""
import pytest

from .test_gpu_prompt_plans import CASES, _cfg
from .test_gpu_prompt_tiles import Case
from .test_host_prompt_tiles import launched


@pytest.mark.parametrize("widths,n,reaches", CASES)
def test_a_case_reaches_the_kernels_it_is_there_for(widths, n, reaches):
    assert reaches <= launched(Case(_cfg(*widths), n, (), chunk=8192))
