"""Numbering, sharing out and cutting of the persistent prefill kernels' tiles (csrc/bm_tile_schedule.h, plain C++; no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, body):
    src = tmp_path / "schedule.cpp"
    src.write_text('#include "bm_tile_schedule.h"\n#include <algorithm>\n#include <cstdio>\n#include <utility>\n#include <vector>\n'
                   '#define CHECK(c, ...) if (!(c)) { std::printf("%s: ", #c); std::printf(__VA_ARGS__); return 1; }\n'
                   'using namespace bm;\nint main() {\n' + body + '  return 0;\n}\n')
    exe = tmp_path / "schedule"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2511_10054_amd", "csrc"), "-o", str(exe), str(src)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_pieces_of_cut_tiles(tmp_path):
    """For every number of tiles of both heights that an XCD can get (and a few more), at reductions from the shortest that are cut on:
    each XCD's tiles follow the one before; the pieces of a tile cover the reduction once, none shorter than 16 k-steps; the
    piece is found again from its first k-step; each piece of a cut tile is one item of one list; their scratch does not overlap and
    ends inside the XCD's; the launch that adds them up has a workgroup row for every cut tile; each number of pieces occurs."""
    _run(tmp_path, r'''
    bool seen[SPLIT_MAX + 1] = {}, seen_small[SPLIT_MAX + 1] = {};
    for (int total : {0, 1, 7, 8, 9, 100, 1000, 4097}) {
        XcdWork w;
        for (int xcd = 0, big = 0; xcd < K64_XCDS; ++xcd, big += w.nb) {
            w.init(total, 3 * total, 64, xcd, false);
            CHECK(w.big0 == big && w.nb >= 0 && w.full == w.nb && w.S == 1, "%d %d\n", total, xcd);
            CHECK(xcd + 1 < K64_XCDS || (w.big0 + w.nb == total && w.small0 + w.ns == 3 * total), "%d\n", total);
        }
    }
    for (int KT : {64, 65, 66, 79, 80, 88, 95, 96, 97, 111, 112, 127, 128, 129, 191, 224, 255, 256, 447, 448, 1024})
        for (int nb = 0; nb <= 100; ++nb)
            for (int ns = 0; ns <= 70; ++ns) {
                XcdWork w, again;
                w.init(nb * K64_XCDS, ns * K64_XCDS, KT, 3, true);
                CHECK(w.nb == nb && w.ns == ns && w.S >= 1 && w.S <= SPLIT_MAX, "%d %d %d\n", KT, nb, ns);
                again.init(nb * K64_XCDS, ns * K64_XCDS, KT, 3, false);
                again.cut(w.S);
                CHECK(again.full == w.full && again.S == w.S, "%d %d %d\n", KT, nb, ns);
                const int R = nb - w.full;
                if (w.S == 1) { CHECK(R == 0, "%d %d %d\n", KT, nb, ns); continue; }
                seen[w.S] |= R > 0;
                seen_small[w.S] |= ns > 0;
                CHECK(R + ns <= FIXUP_TILES && (ns > 0 || R <= FIXUP_TILES_256), "%d %d %d\n", KT, nb, ns);
                int k = 0;
                for (int c = 0; c < w.S; ++c) {
                    int kbeg, kend;
                    w.piece(c, kbeg, kend);
                    CHECK(kbeg == k && kend - kbeg >= 16 && kend - kbeg < KT && w.piece_at(kbeg) == c, "%d %d %d\n", KT, nb, ns);
                    k = kend;
                }
                CHECK(k == KT, "%d %d %d\n", KT, nb, ns);
                std::vector<std::pair<size_t, size_t>> used;
                for (int t = 0; t < R + ns; ++t)
                    for (int c = 0; c < w.S; ++c)
                        used.push_back({w.partial_offset(t, c), w.partial_offset(t, c) + (t < R ? 1 : .5) * SPLIT_TILE_FLOATS});
                std::sort(used.begin(), used.end());
                for (size_t i = 0; i + 1 < used.size(); ++i) CHECK(used[i].second <= used[i + 1].first, "%d %d %d\n", KT, nb, ns);
                CHECK(used.empty() || used.back().second <= (size_t)SPLIT_XCD_TILES * SPLIT_TILE_FLOATS, "%d %d %d\n", KT, nb, ns);
                std::vector<int> items((R + ns) * w.S);
                for (int idx = w.full; idx < w.full + R * w.S; ++idx) {
                    const int c = w.big_piece(idx);
                    const int tile = idx - c * R;
                    CHECK(tile >= w.full && tile < nb && c < w.S, "%d %d %d\n", KT, nb, ns);
                    ++items[(tile - w.full) * w.S + c];
                }
                for (int item = 0; item < ns * w.S; ++item) {
                    const int c = w.small_piece(item);
                    CHECK(c < w.S, "%d %d %d\n", KT, nb, ns);
                    ++items[(R + item - c * ns) * w.S + c];
                }
                for (int n : items) CHECK(n == 1, "%d %d %d\n", KT, nb, ns);
            }
    for (int s = 2; s <= SPLIT_MAX; ++s) CHECK(seen[s] && seen_small[s], "%d pieces\n", s);
''')


def test_column_tiles_of_small_launches(tmp_path):
    """Launches of fewer tiles than units: column tiles cover the matrix once, none wider than the loop that takes it, no more
    tiles than units; from a full launch on everything keeps its width."""
    _run(tmp_path, r'''
    for (int dual = 0; dual < 2; ++dual)
        for (int N = 64; N <= 8192; N += N < 1024 ? 64 : 448)
            for (int n_big = 0; n_big <= 9; ++n_big)
                for (int n_small = 0; n_small <= 260; n_small += 1 + n_small / 7)
                    for (int KT : {4, 5, 6, 40}) {
                        const int n_nt = dual ? (N + 127) / 128 : (N + 255) / 256, n_blk = N / (dual ? 16 : 32), tiles = 2 * n_big + n_small;
                        const SmallPlan p(n_big, n_small, n_nt, n_blk, KT, K64_CUS, true);
                        CHECK(p.cols >= n_nt && p.cols <= n_blk && (p.halved == 0 || p.halved == n_big), "%d %d %d\n", N, n_big, n_small);
                        if (tiles == 0 || tiles * n_nt > K64_CUS) { CHECK(p.cols == n_nt && !p.halved && !p.narrow, "%d %d %d\n", N, n_big, n_small); }
                        else CHECK(p.halved == n_big && tiles * p.cols <= K64_CUS, "%d %d %d\n", N, n_big, n_small);
                        CHECK(!p.narrow || KT >= 6, "%d %d %d\n", N, n_big, n_small);      /* four stages, one tile ahead */
                        for (int ct = 0; ct < p.cols; ++ct) {
                            const int w = (ct + 1) * n_blk / p.cols - ct * n_blk / p.cols;
                            CHECK(w >= 1 && w <= (p.narrow ? 4 : 8), "%d %d %d: %d\n", N, n_big, n_small, w);
                        }
                        const SmallPlan q(n_big, n_small, n_nt, n_blk, KT, K64_CUS, false);
                        CHECK(q.cols == n_nt && !q.halved && !q.narrow, "%d %d %d\n", N, n_big, n_small);
                    }
    for (int n_mt = 1; n_mt <= 13; ++n_mt)
        for (int n_nt = 1; n_nt <= 17; ++n_nt) {
            std::vector<int> hit(n_mt * n_nt);
            for (int id = 0; id < n_mt * n_nt; ++id) {
                int mt, nt;
                tile_of(id, n_mt, n_nt, mt, nt);
                CHECK(mt >= 0 && mt < n_mt && nt >= 0 && nt < n_nt && !hit[mt * n_nt + nt]++, "%d %d %d\n", n_mt, n_nt, id);
            }
        }
''')
