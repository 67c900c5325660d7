"""The build's products: what counts as out of date, and that the library and the module that calls it by address are replaced
together."""
import os
import stat

import pytest

from paper_2411_18462_amd import build


@pytest.fixture
def products(tmp_path, monkeypatch):
    """Stand-ins for everything the build reads and makes, the products a minute younger than the sources."""
    files = {}
    for name, age in (("LIB", 0), ("MARSHAL", 0), ("EXAMPLE_BIN", 0), ("ABI", 60), ("MARSHAL_SRC", 60), ("EXAMPLE_SRC", 60), ("source", 60)):
        p = tmp_path / name
        p.write_text("old")
        os.utime(p, (1e9 - age, 1e9 - age))
        files[name] = p
        if name != "source":
            monkeypatch.setattr(build, name, str(p), raising=False)
    monkeypatch.setattr(build, "SOURCES", [str(files["source"])])
    monkeypatch.setattr(build, "HEADERS", [str(files["ABI"])])
    return files


def test_products_younger_than_their_sources_are_up_to_date(products):
    assert not build.is_stale()


@pytest.mark.parametrize("product,made_from", [("LIB", "source"), ("LIB", "ABI"), ("MARSHAL", "MARSHAL_SRC"), ("MARSHAL", "ABI"),
                                               ("EXAMPLE_BIN", "EXAMPLE_SRC"), ("EXAMPLE_BIN", "ABI")])
def test_a_product_older_than_its_source_is_out_of_date(products, product, made_from):
    """Whatever the age of the other products: a library built after the source changed says nothing about the module."""
    os.utime(products[product], (1e9 - 120, 1e9 - 120))
    assert products[product].stat().st_mtime < products[made_from].stat().st_mtime
    assert build.is_stale()


@pytest.mark.parametrize("product", ["LIB", "MARSHAL", "EXAMPLE_BIN"])
def test_a_missing_product_is_out_of_date(products, product):
    products[product].unlink()
    assert build.is_stale()


def _compiler(path, works):
    """A compiler that writes "new" to its output file, or one that fails after it has."""
    path.write_text("#!/bin/sh\nwhile [ $# -gt 1 ]; do [ \"$1\" = -o ] && printf new > \"$2\"; shift; done\nexit %d\n" % (0 if works else 1))
    path.chmod(path.stat().st_mode | stat.S_IXUSR)
    return str(path)


@pytest.mark.parametrize("hipcc,cxx", [(True, True), (True, False), (False, True)])
def test_library_and_module_are_replaced_together(products, tmp_path, monkeypatch, hipcc, cxx):
    monkeypatch.setenv("HIPCC", _compiler(tmp_path / "hipcc", hipcc))
    monkeypatch.setenv("CXX", _compiler(tmp_path / "cxx", cxx))
    if hipcc and cxx:
        build.build()
    else:
        with pytest.raises(RuntimeError, match="failed"):
            build.build()
    assert {products[p].read_text() for p in ("LIB", "MARSHAL")} == {"new" if hipcc and cxx else "old"}
    assert not [f for f in os.listdir(tmp_path) if ".tmp" in f]
