"""The pool's lookups from the place of the last answer, in any order of questions, without a GPU."""
from test_host_logic import _host_sanitizer_run


def test_lookups_near_the_last_answer(tmp_path):
    _host_sanitizer_run(tmp_path, "pool_lookups", ["ft_pool.cpp"], ["1", "80"], "done 1..80")
