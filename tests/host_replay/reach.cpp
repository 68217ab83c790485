// CPU replay of step-kernel tiles that cross from a cavity's first band into
// its second where a band takes more than a gigabyte, so that a workgroup's
// accesses lie up to two bands from its first block.  The headers check each
// access against the reach of a buffer access.  The state is mapped, not
// allocated: rows far from the boundary stay at rest (zero offsets) and are
// never touched.  One one-step sweep and one K-step launch over the tiles of
// the boundary, in every number of steps and tile shape of the form, must
// equal steps of the 64-bit per-node path bit for bit.
#include <sys/mman.h>

#define main replay_main
#include "replay.cpp"
#undef main

namespace {

template <typename T>
T *mapped(size_t n) {
    void *m = mmap(nullptr, n * sizeof(T), PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) {
        fprintf(stderr, "reach: cannot map %zu bytes\n", n * sizeof(T));
        exit(3);
    }
    return (T *)m;
}

template <int ST>
struct Reach {
    using Lay = typename LayoutOf<ST>::L;
    using R = typename LayoutOf<ST>::R;
    using RH = typename LayoutOf<ST>::RH;
    struct Buf {
        unsigned char *pop;
        R *sr;
    };
    const CavityConst<R> &c;
    Bands bd;
    int xa, xb, ya, yb;  // the window of nodes that are perturbed and advanced
    std::vector<Buf> bufs;
    std::vector<double> acc;

    Buf buf() {
        Buf b{mapped<unsigned char>((size_t)bd.bytes * bd.count), mapped<R>((size_t)c.nx * c.ny)};
        bufs.push_back(b);
        return b;
    }
    void release() {
        for (const Buf &b : bufs) {
            munmap(b.pop, (size_t)bd.bytes * bd.count);
            munmap(b.sr, (size_t)c.nx * c.ny * sizeof(R));
        }
        bufs.clear();
    }
    // One step of the window's nodes at least m nodes inside it, by the 64-bit path.
    void one_step(const Buf &s, const Buf &d, int m) {
        for (int y = ya + m; y < yb - m; ++y)
            for (int x = xa + m; x < xb - m; ++x) step_node<Lay, R, RH, true>(c, s.pop, d.pop, s.sr, d.sr, acc.data(), x, y);
    }
    // The stored populations and source of nodes [x0, x1) x [y0, y1).
    bool same(const Buf &a, const Buf &b, int x0, int x1, int y0, int y1) const {
        const void *pa = band_block(c, (const void *)a.pop, 0), *pb = band_block(c, (const void *)b.pop, 0);
        const AnyBand at_of = any_band(c);
        for (int y = y0; y < y1; ++y)
            for (int x = x0; x < x1; ++x) {
                const FarRef k = at_of(x, y);
                for (int f = 0; f < 3; ++f)
                    for (int i = 0; i < (f == 0 ? 9 : Lay::QT); ++i) {
                        const double va = Lay::template load<RH>(pa, c.band_nodes, f, i, k, c);
                        const double vb = Lay::template load<RH>(pb, c.band_nodes, f, i, k, c);
                        if (std::memcmp(&va, &vb, sizeof(va)) != 0) {
                            printf("differ: field %d direction %d of node (%d, %d)\n", f, i, x, y);
                            return false;
                        }
                    }
                const int64_t q = flat_index(c, x, y);
                if (std::memcmp(&a.sr[q], &b.sr[q], sizeof(R)) != 0) {
                    printf("sources differ at node (%d, %d)\n", x, y);
                    return false;
                }
            }
        return true;
    }

    // the one-step kernel's tile of row y, columns [x0, x1)
    bool row_tile(const Buf &s, const Buf &ref, int y, int x0, int x1) {
        const Buf d = buf();
        const int ba = band_of(c, y - 1);
        const View v = view_of(c, ba, y + 1);
        const NodeConst<R, RH> &n = node_const_of<RH>(c);
        for (int x = x0; x < x1; ++x)
            step_node_view<Lay, R, RH, true>(c, n, true, blocks_of(band_block(c, (const void *)s.pop, ba)),
                                             blocks_of(band_block(c, (const void *)d.pop, ba)), v, s.sr, d.sr, acc.data(),
                                             x, y);
        return same(ref, d, x0, x1, y, y + 1);
    }

    template <int K, int I>
    bool k_tiles(const Buf &s, const Buf &ref, size_t &count) {
        using Tl = StepKTileI<ST, K, I>;
        constexpr int TW = Tl::TW, TH = Tl::TH, NT = Tl::NT;
        using Sh = StepKShape<Lay, TW, TH, K>;
        std::vector<std::pair<int, int>> xs, ys;
        split_runs(c.nx, TW, xs);
        split_runs(c.ny, TH, ys);
        const Buf d = buf();
        for (const auto &yr : ys)
            for (const auto &xr : xs) {
                const int edge = c.band_rows;
                if (yr.first - K >= edge || yr.first + yr.second + K <= edge) continue;  // in one band
                const int cover = K;  // the window's outermost nodes do not hold K steps
                if (xr.first < xa + cover || xr.first + xr.second > xb - cover) continue;
                if (yr.first < ya + cover || yr.first + yr.second > yb - cover) continue;
                const Tile2 tl{0, xr.first, yr.first, xr.second, yr.second};
                std::vector<unsigned char> lds(Sh::LDS_BYTES, 0xff);
                std::vector<R> lds_sr(Sh::NSLOT);
                std::vector<float> lds_b(Sh::STAGE_BASE ? 3 * Sh::NBASE : 1);
                std::memset(lds_sr.data(), 0xff, lds_sr.size() * sizeof(R));
                std::memset(lds_b.data(), 0xff, lds_b.size() * sizeof(float));
                if constexpr (Sh::STAGE_BASE)
                    for (int t = 0; t < NT; ++t)
                        stepk_stage_bases<Lay, R, TW, TH, K, NT>(c, tl, s.pop, lds_b.data(), t);
                for (int t = 0; t < NT; ++t)
                    if (t < Sh::LW * (tl.h + 2 * Sh::RING))
                        stepk_first<Lay, R, RH, TW, TH, K>(c, tl, s.pop, s.sr, acc.data(), lds.data(), lds_sr.data(),
                                                           lds_b.data(), t);
                for (int j = K - 2; j >= 1; --j) {
                    std::vector<MidNode<R, RH>> nodes(NT);
                    std::vector<char> act(NT, 0);
                    for (int t = 0; t < NT; ++t)
                        act[t] = t < (TW + 2 * j) * (tl.h + 2 * j) &&
                                 stepk_mid_load<Lay, R, RH, TW, TH, K>(c, tl, j, lds.data(), lds_sr.data(), t, nodes[t]);
                    for (int t = 0; t < NT; ++t)
                        if (act[t])
                            stepk_mid_store<Lay, R, RH, TW, TH, K>(c, tl, acc.data(), lds.data(), lds_sr.data(), nodes[t]);
                }
                for (int t = 0; t < NT; ++t)
                    if (t < TW * tl.h)
                        stepk_last<Lay, R, RH, TW, TH, K>(c, tl, d.pop, d.sr, acc.data(), lds.data(), lds_sr.data(), t);
                if (!same(ref, d, tl.x0, tl.x0 + tl.w, tl.y0, tl.y0 + tl.h)) return false;
                ++count;
            }
        return true;
    }
};

template <int ST>
int check(const Job &j) {
    using Rc = Reach<ST>;
    using R = typename Rc::R;
    using RH = typename Rc::RH;
    Lattice l;
    if (map_params(j.p, j.prec, l) != LBM_OK) {
        fprintf(stderr, "reach: %s\n", g_err);
        return 2;
    }
    const int nx = j.p.nx, ny = j.p.ny;
    const Bands bd = bands_of(nx, ny, Rc::Lay::bytes_per_node, 0, j.p.band_rows);
    if (bd.nodes * (Rc::Lay::bytes_per_node + 8) >= ((int64_t)1 << 31)) return 2;  // as the plan refuses
    const CavityConst<R> c = make_const<R>(l, 0, 0, bd);
    // the last columns, where a plane's offsets are largest, around the boundary
    Rc r{c, bd, nx - 150, nx - 10, std::max(10, bd.rows - 40), std::min(ny - 10, bd.rows + 40), {}, {}};
    r.acc.assign((size_t)4 * ((size_t)nx + ny), 0.0);
    size_t tiles = 0;
    auto start = [&]() {
        const typename Rc::Buf s = r.buf();
        uint64_t seed = j.seed;
        for (int y = r.ya - 4; y < r.yb + 4; ++y)
            for (int x = r.xa - 4; x < r.xb + 4; ++x)
                init_node<typename Rc::Lay, R, RH>(c, s.pop, s.sr, x, y, j.p.T_init + 1e5 * noise(seed), j.p.T_init);
        return s;
    };
    auto shapes = [&](auto kk) -> bool {
        constexpr int K = decltype(kk)::value;
        const typename Rc::Buf s = start();
        std::vector<typename Rc::Buf> steps{s};
        for (int q = 0; q < K; ++q) {
            steps.push_back(r.buf());
            r.one_step(steps[q], steps[q + 1], q);
        }
        bool ok = true;
        if (K == 2)
            for (int y = bd.rows - 2; y < bd.rows + 2 && ok; ++y) ok = r.row_tile(s, steps[1], y, r.xa + 1, r.xb - 1);
        ok = ok && r.template k_tiles<K, 0>(s, steps[K], tiles);
        if constexpr (stepk_offered(ST, K)) {
            ok = ok && r.template k_tiles<K, 1>(s, steps[K], tiles);
            ok = ok && r.template k_tiles<K, 2>(s, steps[K], tiles);
        }
        r.release();
        return ok;
    };
    if (!shapes(std::integral_constant<int, 2>{}) || !shapes(std::integral_constant<int, 3>{})) return 1;
    printf("identical: %zu tiles, %d bands of %lld bytes\n", tiles, bd.count, (long long)bd.bytes);
    return 0;
}

}  // namespace

int main() {
    Job j;
    if (!read_job(j)) return 2;
    switch (storage_of(j.prec, j.p.thermal_lattice == 5 ? 5 : 9)) {
        case ST_F64: return check<ST_F64>(j);
        case ST_F32: return check<ST_F32>(j);
        case ST_F32H: return check<ST_F32H>(j);
        case ST_F16: return check<ST_F16>(j);
        case ST_F16S: return check<ST_F16S>(j);
        case ST5_F64: return check<ST5_F64>(j);
        case ST5_F32: return check<ST5_F32>(j);
    }
    return 2;
}
