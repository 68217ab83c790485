// CPU replay of the deep launches, with the state, one-step path and job
// format of replay.cpp: every thread's load, then per update every thread's
// update, LDS write and LDS read in the kernel's barrier order, then the
// stores.  The LDS of each emulated workgroup is as large as the kernel's and
// filled with NaN bit patterns.  For every number of steps a launch of the
// shape takes (shape of the job, `launches` launches of each), the state must
// equal that of single steps bit for bit.
#define main replay_main
#include "replay.cpp"
#undef main

namespace {

template <int ST, int I>
void deep_all(const CavityConst<typename LayoutOf<ST>::R> &c, State<ST> &S, int cur, const std::vector<Tile2> &tiles,
              int k) {
    using Lay = typename LayoutOf<ST>::L;
    using R = typename LayoutOf<ST>::R;
    using RH = typename LayoutOf<ST>::RH;
    constexpr DeepDims d = deep_dims(ST, I);
    using Sh = DeepShape<Lay, d.tw, d.th, d.k>;
    const NodeConst<R, RH> &n = node_const_of<RH>(c);
    for (const Tile2 &tl : tiles) {
        std::vector<unsigned char> lds(Sh::LDS_BYTES, 0xff);
        const TileView<R> tv = tile_view<Sh>(c, tl);
        std::vector<DeepNode<R, RH>> q(Sh::NT);
        std::vector<char> act(Sh::NT);
        for (int t = 0; t < Sh::NT; ++t)
            deep_load<Sh, Lay, R, RH>(tv, n, S.pop[cur].data(), S.sr[cur].data(), S.acc.data(), k, t, q[t]);
        for (int left = k - 1;; --left) {
            for (int t = 0; t < Sh::NT; ++t) act[t] = deep_update<Sh, R, RH>(tv, n, left, q[t]);
            if (left == 0) break;
            for (int t = 0; t < Sh::NT; ++t)
                if (act[t]) deep_put<Sh, R, RH>(n, lds.data(), t, q[t]);
            for (int t = 0; t < Sh::NT; ++t) deep_pull<Sh, R, RH>(n, lds.data(), left - 1, q[t]);
        }
        for (int t = 0; t < Sh::NT; ++t)
            deep_store<Sh, Lay, R, RH>(tv, n, S.pop[1 - cur].data(), S.sr[1 - cur].data(), S.acc.data(), q[t]);
    }
}

template <int ST, int I>
int check(const Job &j) {
    using Lay = typename LayoutOf<ST>::L;
    using R = typename LayoutOf<ST>::R;
    using RH = typename LayoutOf<ST>::RH;
    Lattice l;
    if (map_params(j.p, j.prec, l) != LBM_OK) {
        fprintf(stderr, "deep: %s\n", g_err);
        return 2;
    }
    const int nx = j.p.nx, ny = j.p.ny;
    const Bands bd = bands_of(nx, ny, Lay::bytes_per_node, 0, j.p.band_rows);
    const CavityConst<R> c = make_const<R>(l, 0, 0, bd);
    State<ST> A;
    const size_t pop_bytes = (size_t)bd.bytes * bd.count, nodes = (size_t)nx * ny;
    for (int b = 0; b < 2; ++b) {
        A.pop[b].assign(pop_bytes, 0);
        A.sr[b].assign(nodes, R(0));
    }
    A.acc.assign((size_t)4 * (nx + ny), 0.0);
    uint64_t s = j.seed;
    for (int y = 0; y < ny; ++y)
        for (int x = 0; x < nx; ++x)  // solid, mushy and liquid nodes
            init_node<Lay, R, RH>(c, A.pop[0].data(), A.sr[0].data(), x, y, j.p.T_init + 1e5 * noise(s), j.p.T_init);
    one_step_all<ST>(c, A, 0, false);
    constexpr DeepDims d = deep_dims(ST, I);
    std::vector<Tile2> tiles;
    cavity_tiles2(0, nx, ny, d.tw, d.th, tiles);
    State<ST> B = A;
    int ca = 1, cb = 1;
    for (int k = d.k; k >= 2; --k)
        for (int launch = 0; launch < j.launches; ++launch) {
            for (int q = 0; q < k; ++q) {
                one_step_all<ST>(c, A, ca, true);
                ca ^= 1;
            }
            deep_all<ST, I>(c, B, cb, tiles, k);
            cb ^= 1;
            if (std::memcmp(A.pop[ca].data(), B.pop[cb].data(), pop_bytes) != 0 ||
                std::memcmp(A.sr[ca].data(), B.sr[cb].data(), nodes * sizeof(R)) != 0 ||
                std::memcmp(A.acc.data(), B.acc.data(), A.acc.size() * sizeof(double)) != 0) {
                printf("differ: %d steps, tiles of %dx%d\n", k, d.tw, d.th);
                return 1;
            }
        }
    for (double v : A.acc)
        if (!(v == v)) {
            printf("tallies hold NaN\n");
            return 1;
        }
    printf("identical\n");
    return 0;
}

template <int ST>
int run_shape(const Job &j) {
    static_assert(kDeepShapes == 4, "one case per shape");
    switch (j.shape) {
        case 0: return check<ST, 0>(j);
        case 1: return check<ST, 1>(j);
        case 2: return check<ST, 2>(j);
        case 3: return check<ST, 3>(j);
    }
    return 2;
}

}  // namespace

int main() {
    Job j;
    if (!read_job(j)) return 2;
    switch (storage_of(j.prec, j.p.thermal_lattice == 5 ? 5 : 9)) {
        case ST_F64: return run_shape<ST_F64>(j);
        case ST_F32: return run_shape<ST_F32>(j);
        case ST_F32H: return run_shape<ST_F32H>(j);
        case ST5_F64: return run_shape<ST5_F64>(j);
        case ST5_F32: return run_shape<ST5_F32>(j);
        case ST5_F32H: return run_shape<ST5_F32H>(j);
    }
    return 2;
}
