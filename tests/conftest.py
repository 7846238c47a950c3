import ctypes
import os
import subprocess
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def _gpu_available() -> bool:
    try:
        import torch
        return torch.cuda.is_available()
    except Exception:
        return False


def pytest_collection_modifyitems(config, items):
    if _gpu_available():
        return
    skip = pytest.mark.skip(reason="no GPU in this container")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


PLAN_SOURCE = """
#include "prefix_plan.h"
extern "C" {
// out: symbols compared in registers, kind or size, groups, threads, lanes, row_bytes, body, hash_groups, total, LDS of a workgroup
static void layout(const sr::PrefixGeom &q, bool direct, int size, int lds, int *out) {
    const int v[] = {direct, size, q.groups, q.threads, q.lanes, q.row_bytes, q.body, q.hash_groups, q.total, lds};
    for (int i = 0; i < 10; ++i) out[i] = v[i];
}
int gate_layout(int n_groups, int G, int L, int *out) {
    sr::GateLayout t;
    if (!sr::gate_layout(n_groups, G, L, &t)) return 0;
    layout(t.q, t.direct, t.size, t.lds, out);
    return 1;
}
int signals_layout(int n_groups, int G, int L, int n_lens, int distinct, int *out) {
    sr::SignalsLayout t;
    if (!sr::signals_layout(n_groups, G, L, n_lens, distinct, &t)) return 0;
    layout(t.q, t.direct, t.size, t.lds, out);
    return 1;
}
// turns of a full workgroup of that layout (n_lens = 0: the gate's): hashed, groups of a turn, bytes of a group's tables
void prefix_turns(int n_groups, int G, int L, int n_lens, unsigned most, int *out) {
    sr::GateLayout g;
    sr::SignalsLayout s;
    if (n_lens) sr::signals_layout(n_groups, G, L, n_lens, n_lens, &s);
    else sr::gate_layout(n_groups, G, L, &g);
    const sr::PrefixGeom &q = n_lens ? s.q : g.q;
    const sr::PrefixTurns t = sr::prefix_turns(q, q.groups, most);
    out[0] = t.hashed; out[1] = t.groups; out[2] = t.group_bytes;
}
void shared_tiles(int n_sets, int per_set, int *set, int *part) {
    for (int wg = 0; wg < n_sets * per_set; ++wg) sr::shared_tiles_of(wg, n_sets, per_set, set + wg, part + wg);
}
int divide(int n, int d) { return sr::quotient(n, sr::fast_div(d)); }
int stream_waves(int M, int N, int ks, int swiglu) { return sr::stream_waves(M, N, ks, swiglu); }
int plan_kernel(int M, int N, int ks, int mt_total, int swiglu, int splits) {
    return sr::plan_gemm(M, N, ks, mt_total, swiglu, splits, 16).kernel;
}
int tile_nt(int i) { return sr::kTileShapes[i].nt; }
int tile_rt(int i) { return sr::kTileShapes[i].rt; }
int split_steps(int M, int N, int ks, int mt_total, int splits) { return sr::split_steps(M, N, ks, mt_total, splits); }
int score_rows(int M, int vocab, int rows) { return sr::score_rows(M, vocab, rows); }
int private_splits(int waves1, int shared_waves, int tokens, int most) { return sr::private_splits(waves1, shared_waves, tokens, most); }
int token_splits(int tokens, int want, int *each) { const sr::TokenSplits s = sr::token_splits(tokens, want); *each = s.tokens; return s.n; }
int whole_context(int n_kv, int head_dim, int ctx, int groups, int G, int shared) {
    return sr::whole_context((long long)groups * G, n_kv, head_dim, ctx, groups, G, shared);
}
int thin_resid(int M, int N, int ks) { return sr::thin_resid(M, N, ks); }
int thin_qkv(int M, int N, int ks) { return sr::thin_qkv(M, N, ks); }
void rope_tables(int len, int d, double theta, float *c, float *s) { sr::rope_tables(len, d, theta, c, s); }
int padded_k_steps(int K) { return sr::padded_k_steps(K); }
int projection_splits(int M, int N, int ks, int mt_total) { return sr::projection_splits(M, N, ks, mt_total); }
int stream_lean(int M, int wide, int ks, int splits, int scaled) { return sr::stream_lean(M, wide, ks, splits, scaled); }
int plan_projection(int M, int N, int ks, int mt_total, int swiglu, int max_splits, int *out) {
    const sr::ProjectionPlan p = sr::plan_projection(M, N, ks, mt_total, swiglu, max_splits);
    out[0] = p.nt; out[1] = p.rt; out[2] = p.splits;
    return p.wide;
}
// first k-step of every split of that plan, and the end of the last
void split_ranges(int M, int N, int ks, int mt_total, int swiglu, int max_splits, int *from) {
    const sr::ProjectionPlan p = sr::plan_projection(M, N, ks, mt_total, swiglu, max_splits);
    for (int sp = 0; sp < p.splits; ++sp) sr::split_range(ks, p.steps, p.splits, sp, from + sp, from + sp + 1);
}
}
"""


@pytest.fixture(scope="session")
def plan(tmp_path_factory):
    """csrc/plan.h as a shared library: which kernel a projection runs on.  plan.kernel(rows, matrix rows, inner dimension,
    swiglu, splits) names it for a context of up to 8192 rows per pass, so that a test can say what it means to reach."""
    from paper_2605_05802_amd.build import CSRC
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PLAN_SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(d / "plan.cpp"), "-o", str(d / "plan.so")])
    lib = ctypes.CDLL(str(d / "plan.so"))

    def kernel(M, N, K, swiglu=False, splits=1):
        ks = lib.padded_k_steps(K)
        waves = lib.stream_waves(M, N, ks, int(swiglu))
        if waves:
            return f"stream {waves}"
        k = lib.plan_kernel(M, N, ks, 512, int(swiglu), splits)
        if k >= 0:
            return f"tiles {lib.tile_nt(k)}x{lib.tile_rt(k)}"
        return "128" if k == -2 else "rows16" if M <= 384 else "rows32"

    def projection(M, N, K, swiglu=False, max_splits=1):
        """The final choice, (kernel, K splits): deep projections of a few hundred rows have tile shapes that the others have not."""
        ks, out = lib.padded_k_steps(K), (ctypes.c_int * 3)()
        lib.plan_projection(M, N, ks, 512, int(swiglu), max_splits, out)
        return (f"tiles {out[0]}x{out[1]}" if out[0] else kernel(M, N, K, swiglu, out[2])), out[2]

    lib.kernel = kernel
    lib.projection = projection
    return lib
