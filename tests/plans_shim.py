"""The host's launch rules (csrc/plans.h), compiled for the CPU tests."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "plans.h"
#include <string.h>
using namespace swdb;
static Matrix mat_of(const int8_t* v) { Matrix m; memcpy(m.v, v, sizeof(m.v)); return m; }
extern "C" {
// {group, guard, c2, ge2, group2, lim2, over2}
void p_drift(int m, int64_t cols, int R, const int8_t* v, int go, int ge, int limit,
             int64_t short_cols, uint32_t* out) {
  const DriftArgs d = drift_plan(m, cols, R, mat_of(v), go, ge, limit, short_cols);
  const uint32_t r[7] = {(uint32_t)d.group, (uint32_t)d.guard, d.c2, d.ge2, d.group2, d.lim2, d.over2};
  memcpy(out, r, sizeof(r));
}
// {add, bias, top, top_byte, code_byte, row_byte}
static void put(const PairForm& f, int32_t* out) {
  const int32_t r[6] = {f.add, f.bias, f.top, f.top_byte, f.code_byte, f.row_byte};
  memcpy(out, r, sizeof(r));
}
void p_pair(const int8_t* v, int ge, int limit, int32_t* out) { put(pair_form(mat_of(v), ge, limit), out); }
// {R, W, strips, base, pad}
void p_mode(int m, int64_t cols, const int8_t* v, int go, int ge, int mode, int32_t* out) {
  const ModePlan p = mode_plan(m, cols, mat_of(v), go, ge, mode);
  const int32_t r[5] = {p.R, p.W, p.n_strips, p.shape.base, p.shape.pad};
  memcpy(out, r, sizeof(r));
}
// {form, base, pad}
void p_mode_pairs(int m, int64_t longest, const int8_t* v, int go, int ge, int mode, int R,
                  int32_t* out) {
  ModeShape s{};
  put(mode_pairs(m, longest, mat_of(v), go, ge, mode, R, &s), out);
  out[6] = s.base;
  out[7] = s.pad;
}
// {ring, grid, rows}
void p_rows(int ring, int grid, int n_pass, int64_t items, int64_t stride, int64_t have, int64_t* out) {
  const PairRows r = pair_rows(ring, grid, n_pass, items, stride, have);
  out[0] = r.ring;
  out[1] = r.grid;
  out[2] = r.rows;
}
// {R, W, grid}
void p_launch(int m, const double* d, const int64_t* bins, int64_t n_bins, int cus, int rows,
              int waves, int own, int32_t* out) {
  PairLoad p;
  p.bins = bins;
  p.n_bins = n_bins;
  p.bin_col = std::max(m * 128 / 4.5e10, 2.5e-7);
  p.m = m;
  p.items = d[0];
  p.cols = d[1];
  p.longest = d[2];
  p.beside = d[3];
  p.cus = cus;
  p.rows = rows;
  p.waves = waves;
  p.own = own != 0;
  const PairLaunch l = pair_launch(p);
  out[0] = l.R;
  out[1] = l.W;
  out[2] = l.grid;
}
int p_batch(const int64_t* lens, int64_t n, const double* d, int cus, int rows, int waves, int32_t* rw) {
  return batch_schedule(lens, n, d[0], d[1], cus, rows, waves, rw, rw + 1);
}
void p_half(int m, const double* d, int32_t* rw) { half_rows(m, d[0], d[1], d[2], rw, rw + 1, d[3]); }
int p_lds(int R, int W, int n_pass, int own) {
  const size_t mine = pairs_lds(R, W, n_pass, false), all = pairs_lds(R, W, n_pass, true);
  return (int)((own ? mine : std::min(mine, all)) + pairs_lds_static(W));
}
int p_ring(int n_pass, int W) { return pair_ring(n_pass, W); }
}
"""
_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as tmp:
            src, so = os.path.join(tmp, "shim.cpp"), os.path.join(tmp, "shim.so")
            with open(src, "w") as f:
                f.write(SHIM)
            subprocess.check_call(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wall", "-I",
                                   os.path.join(ROOT, "paper_2203_11100_amd", "csrc"), src, "-o",
                                   so])
            _lib = ctypes.CDLL(so)
    return _lib


def _mat(matrix):
    return np.ascontiguousarray(matrix, dtype=np.int8).ctypes.data_as(ctypes.c_void_p)


def _i64(v):
    return ctypes.c_int64(int(v))


def drift(m, cols, R, matrix, go, ge, limit=32767, short_cols=0):
    out = np.zeros(7, np.uint32)
    lib().p_drift(m, _i64(cols), R, _mat(matrix), go, ge, limit, _i64(short_cols),
                  out.ctypes.data_as(ctypes.c_void_p))
    return dict(zip(("group", "guard", "c2", "ge2", "group2", "lim2", "over2"), out.tolist()))


PAIR = ("add", "bias", "top", "top_byte", "code_byte", "row_byte")


def pair(matrix, ge, limit=32767):
    out = np.zeros(6, np.int32)
    lib().p_pair(_mat(matrix), ge, limit, out.ctypes.data_as(ctypes.c_void_p))
    return dict(zip(PAIR, out.tolist()))


def mode(m, cols, matrix, go, ge, mode):
    out = np.zeros(5, np.int32)
    lib().p_mode(m, _i64(cols), _mat(matrix), go, ge, mode, out.ctypes.data_as(ctypes.c_void_p))
    return dict(zip(("R", "W", "strips", "base", "pad"), out.tolist()))


def mode_pairs(m, longest, matrix, go, ge, mode, R):
    out = np.zeros(8, np.int32)
    lib().p_mode_pairs(m, _i64(longest), _mat(matrix), go, ge, mode, R,
                       out.ctypes.data_as(ctypes.c_void_p))
    return dict(zip(PAIR + ("base", "pad"), out.tolist()))


def rows(n_pass, W, grid, items, stride, have=-1):
    out = np.zeros(3, np.int64)
    lib().p_rows(lib().p_ring(n_pass, W), grid, n_pass, _i64(items), _i64(stride), _i64(have),
                 out.ctypes.data_as(ctypes.c_void_p))
    return dict(zip(("ring", "grid", "rows"), out.tolist()))


def launch(m, items, cols, longest, beside=0.0, cus=256, rows=0, waves=0, own=False, bins=()):
    out = np.zeros(3, np.int32)
    desc = np.zeros((len(bins) + 1, 4), np.int64)
    desc[:len(bins), 2] = bins
    d = np.array([items, cols, longest, beside], np.float64)
    lib().p_launch(m, d.ctypes.data_as(ctypes.c_void_p), desc.ctypes.data_as(ctypes.c_void_p),
                   _i64(len(bins)), cus, rows, waves, int(own),
                   out.ctypes.data_as(ctypes.c_void_p))
    return tuple(out.tolist())


def lds(R, W, n_pass, own=False):
    return lib().p_lds(R, W, n_pass, int(own))


def half_rows(m, items, cols, longest, rows, waves, beside=0.0):
    rw, d = np.array([rows, waves], np.int32), np.array([items, cols, longest, beside], np.float64)
    lib().p_half(m, d.ctypes.data_as(ctypes.c_void_p), rw.ctypes.data_as(ctypes.c_void_p))
    return tuple(rw.tolist())


def batch(lens, cols, longest, cus=256, rows=0, waves=0):
    rw, d = np.zeros(2, np.int32), np.array([cols, longest], np.float64)
    v = np.array(sorted(lens, reverse=True), np.int64)
    ok = lib().p_batch(v.ctypes.data_as(ctypes.c_void_p), _i64(len(v)),
                       d.ctypes.data_as(ctypes.c_void_p), cus, rows, waves,
                       rw.ctypes.data_as(ctypes.c_void_p))
    return tuple(rw.tolist()) if ok else None
