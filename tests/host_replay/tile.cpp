// CPU replay of the multi-step kernels with their wall tallies in LDS, which
// replay.cpp keeps in the cavity's memory: every tile's LDS tallies start as
// NaN and are as large as the kernel's, so a slot that the first update does not
// fill, or that another tile's node reads, shows in the result.  The idle
// threads' fetches for each tile run too, for their addresses (the state's
// buffers end with the state).  State, sources and tallies must equal single
// steps bit for bit.
#define main replay_main
#include "replay.cpp"
#undef main

namespace {

template <int ST, int K, int I>
bool tiles_all(const CavityConst<typename LayoutOf<ST>::R> &c, State<ST> &S, int cur, const std::vector<Tile2> &tiles) {
    using Lay = typename LayoutOf<ST>::L;
    using R = typename LayoutOf<ST>::R;
    using RH = typename LayoutOf<ST>::RH;
    using Tl = StepKTileI<ST, K, I>;
    constexpr int TW = Tl::TW, TH = Tl::TH, NT = Tl::NT, BUSY = (TW * TH + 63) / 64 * 64;
    using Sh = StepKShape<Lay, TW, TH, K>;
    using InTile = typename std::conditional<Sh::TILE_TALLY, TileTally<TW, TH, false, R>, CavityTally<double, R>>::type;
    using InLast = typename std::conditional<Sh::TILE_TALLY, TileTally<TW, TH, true, R>, CavityTally<double, R>>::type;
    const NodeConst<R, RH> &n = node_const_of<RH>(c);
    const CavityTally<double, R> all{S.acc.data(), c};
    for (const Tile2 &tl : tiles) {
        std::vector<unsigned char> lds(Sh::LDS_BYTES, 0xff);
        std::vector<R> lds_sr(Sh::NSLOT);
        std::memset(lds_sr.data(), 0xff, lds_sr.size() * sizeof(R));
        std::vector<float> lds_b(Sh::STAGE_BASE ? 3 * Sh::NBASE : 1);
        std::vector<double> lds_t(Sh::TILE_TALLY ? 4 * (TW + TH) : 1);
        std::memset(lds_t.data(), 0xff, lds_t.size() * sizeof(double));
        const TileView<R> tv = tile_view<Sh>(c, tl);
        const InTile tally = tally_of<InTile>(all, lds_t.data(), tv);
        const InLast last = tally_of<InLast>(all, lds_t.data(), tv);
        const void *src = S.pop[cur].data();
        if constexpr (Sh::STAGE_BASE)
            for (int t = 0; t < NT; ++t) stepk_stage_bases<Lay, R, TW, TH, K, NT>(tv, src, lds_b.data(), t);
        for (int t = 0; t < NT; ++t)
            if (t < Sh::LW * (tl.h + 2 * Sh::RING))
                stepk_first<Lay, R, RH, TW, TH, K>(tv, n, src, S.sr[cur].data(), tally, lds.data(), lds_sr.data(),
                                                   lds_b.data(), t);
        if constexpr (K == 3) {
            std::vector<MidNode<R, RH>> nodes(NT);
            std::vector<char> act(NT, 0);
            for (int t = 0; t < NT; ++t)
                act[t] = t < (TW + 2) * (tl.h + 2) &&
                         stepk_mid_load<Lay, R, RH, TW, TH, K, 1>(tv, n, lds.data(), lds_sr.data(), t, nodes[t]);
            for (int t = 0; t < NT; ++t)
                if (act[t])
                    stepk_mid_store<Lay, R, RH, TW, TH, K, 1>(tv, n, tally, lds.data(), lds_sr.data(), nodes[t]);
        }
        for (int t = 0; t < NT; ++t)
            if (t < TW * tl.h)
                stepk_last<Lay, R, RH, TW, TH, K>(tv, n, S.pop[1 - cur].data(), S.sr[1 - cur].data(), last, lds.data(),
                                                  lds_sr.data(), t);
        if constexpr (K == 3 && NT > BUSY)
            for (int t = 0; t < NT - BUSY; ++t) stepk_prefetch<Lay, R, TW, TH, K, NT - BUSY>(c, tl, src, t);
    }
    return Sh::TILE_TALLY;
}

template <int ST, int K, int I>
int check(const Job &j) {
    using Lay = typename LayoutOf<ST>::L;
    using R = typename LayoutOf<ST>::R;
    using RH = typename LayoutOf<ST>::RH;
    Lattice l;
    if (map_params(j.p, j.prec, l) != LBM_OK) {
        fprintf(stderr, "tile: %s\n", g_err);
        return 2;
    }
    const int nx = j.p.nx, ny = j.p.ny;
    const Bands bd = bands_of(nx, ny, Lay::bytes_per_node, 0, j.p.band_rows);
    const CavityConst<R> c = make_const<R>(l, 0, 0, bd);
    const size_t pop_bytes = (size_t)bd.bytes * bd.count, nodes = (size_t)nx * ny;
    State<ST> A;
    for (int b = 0; b < 2; ++b) {
        A.pop[b].assign(pop_bytes, 0);
        A.sr[b].assign(nodes, R(0));
    }
    A.acc.assign((size_t)4 * (nx + ny), 0.0);
    uint64_t s = j.seed;
    for (int y = 0; y < ny; ++y)
        for (int x = 0; x < nx; ++x)
            init_node<Lay, R, RH>(c, A.pop[0].data(), A.sr[0].data(), x, y, j.p.T_init + 1e5 * noise(s), j.p.T_init);
    one_step_all<ST>(c, A, 0, false);
    std::vector<Tile2> tiles;
    cavity_tiles2(0, nx, ny, dims_of<ST, K>(I).tw, dims_of<ST, K>(I).th, tiles);
    State<ST> B = A;
    int ca = 1, cb = 1;
    bool in_lds = false;
    for (int launch = 0; launch < j.launches; ++launch) {
        for (int q = 0; q < K; ++q, ca ^= 1) one_step_all<ST>(c, A, ca, true);
        in_lds = tiles_all<ST, K, I>(c, B, cb, tiles);
        cb ^= 1;
    }
    if (std::memcmp(A.pop[ca].data(), B.pop[cb].data(), pop_bytes) != 0 ||
        std::memcmp(A.sr[ca].data(), B.sr[cb].data(), nodes * sizeof(R)) != 0 ||
        std::memcmp(A.acc.data(), B.acc.data(), A.acc.size() * sizeof(double)) != 0) {
        printf("differ: %d steps, tile shape %d\n", K, I);
        return 1;
    }
    for (double v : A.acc)
        if (!(v == v)) {
            printf("tallies hold NaN\n");
            return 1;
        }
    printf("identical, tallies in %s\n", in_lds ? "LDS" : "memory");
    return 0;
}

template <int ST>
int run_form(const Job &j) {
    if (j.K == 2) {
        if (j.shape == 0) return check<ST, 2, 0>(j);
        if (j.shape == 1) return check<ST, 2, 1>(j);
        return check<ST, 2, 2>(j);
    }
    if (j.shape == 0) return check<ST, 3, 0>(j);
    if constexpr (stepk_offered(ST, 3)) {
        if (j.shape == 1) return check<ST, 3, 1>(j);
        return check<ST, 3, 2>(j);
    }
    return 2;
}

}  // namespace

int main() {
    Job j;
    if (!read_job(j)) return 2;
    switch (storage_of(j.prec, j.p.thermal_lattice == 5 ? 5 : 9)) {
        case ST_F64: return run_form<ST_F64>(j);
        case ST_F32: return run_form<ST_F32>(j);
        case ST_F32H: return run_form<ST_F32H>(j);
        case ST_F16: return run_form<ST_F16>(j);
        case ST_F16S: return run_form<ST_F16S>(j);
        case ST5_F64: return run_form<ST5_F64>(j);
        case ST5_F32: return run_form<ST5_F32>(j);
        case ST5_F32H: return run_form<ST5_F32H>(j);
    }
    return 2;
}
