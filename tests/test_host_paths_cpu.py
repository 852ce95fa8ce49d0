"""The library's host side without a GPU: sizes of workspaces, fall-backs when
memory runs out, memory budgets and graph captures, on a HIP runtime in host
memory whose kernels are logged and not run."""
import pytest

from tests import host_hip


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = host_hip.build(tmp_path_factory.mktemp("host_hip"))
    return lambda case, **kw: host_hip.run(so, "tests.host_cases", case, **kw)


def test_gradient_partial_sums_fit_what_larger_batches_reserved(host):
    host("gradient_parts")


def test_stream_graph_holds_every_tile_after_steps_without_it(host):
    host("stream_graph_switched_on_and_off")


@pytest.mark.parametrize("how", ["set", "load"])
def test_forced_row_shape_after_the_default(host, how, tmp_path):
    host("forced_shape_after_default", how=how if how == "set" else str(tmp_path))


@pytest.mark.parametrize("case", ["stream_budget", "stream_budget_with_worker", "stream_without_room_for_tables"])
def test_stream_keeps_its_memory_budget(host, case):
    host(case)


def test_default_row_shape_without_room_for_its_tables(host):
    host("row_tables_without_room")


def test_mitigation_without_room_for_split_sums(host):
    host("rfi_without_room_for_sums")


def test_network_after_a_batch_without_room(host):
    host("network_after_a_batch_without_room")


def test_stream_rows_of_one_round_take_the_pattern_tile(host):
    host("stream_rows_of_one_round")
