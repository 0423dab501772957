// The listing of steps (host.cpp) at every width, chunk length and piece length that a plan can have: every leaf is listed once, at the place and with the row
// of C of its fiber, and chunks, groups and slices are counted as the kernels count them.  Exit code 0 when all hold; prints the first that does not.
#include "../../paper_2311_09549_amd/csrc/host.cpp"

#include <random>

struct Tensor {
    std::vector<int32_t> pos[3], crd[3], fiber_of, slice_of;
    int64_t nfib[4] = {0, 0, 0, 0};
    HostCsf view() const
    {
        HostCsf h;
        for (int m = 0; m < 3; ++m) {
            h.crd[m] = crd[m].data();
            h.pos[m] = pos[m].data();
        }
        h.have_crd = true;
        return h;
    }
    Tensor(const std::vector<std::vector<int>> &shape, std::mt19937 &rng)   // fiber lengths per slice
    {
        pos[1] = pos[2] = {0};
        for (const auto &slice : shape) {
            crd[0].push_back((int32_t)crd[0].size());
            for (int len : slice) {
                slice_of.push_back((int32_t)crd[0].size() - 1);
                crd[1].push_back((int32_t)(rng() % 10000));
                for (int n = 0; n < len; ++n) {
                    fiber_of.push_back((int32_t)crd[1].size() - 1);
                    crd[2].push_back((int32_t)(rng() % 10000));
                }
                pos[2].push_back((int32_t)crd[2].size());
            }
            pos[1].push_back((int32_t)crd[1].size());
        }
        for (int m = 0; m < 3; ++m) nfib[m] = (int64_t)crd[m].size();
    }
};

// 0, or the line of the check that failed
static int check(const Tensor &t, SliceSource src, int R, sc_dtype dtype, int piece, int cap, int tune)
{
#define REQUIRE(x) do { if (!(x)) return __LINE__; } while (0)
    sc_plan p{};
    p.kind = src == SLICE_MTTKRP ? K_MTTKRP3 : K_TTMC3;
    p.dtype = dtype;
    p.order = 3;
    p.nnz = t.nfib[2];
    for (int m = 0; m < 4; ++m) p.nfib[m] = t.nfib[m];
    p.fcols[0] = p.fcols[1] = R;
    p.sched = piece == 1 ? SC_SCHED_LINEAR : SC_SCHED_FUSED;
    p.tune.tn = tune;
    const int wide = src == SLICE_MTTKRP ? 1024 / (R * (int)esize(dtype)) : 4;
    p.n_cu = cap ? std::max<int64_t>(1, p.nnz / ((int64_t)wide * cap * 8)) : 1 << 30;   // chunks of `cap` steps, or the shortest there are
    const HostCsf h = t.view();
    SliceBuild b;
    build_slices(&p, src, piece, h, b);

    std::vector<uint32_t> leaf, at;
    std::vector<int32_t> gj;
    for (const SlicePart &q : b.parts) {
        leaf.insert(leaf.end(), q.leaf.begin(), q.leaf.end());
        at.insert(at.end(), q.at.begin(), q.at.end());
        gj.insert(gj.end(), q.gj.begin(), q.gj.end());
    }
    REQUIRE(leaf.size() == 4 * at.size());
    const uint8_t *place = reinterpret_cast<const uint8_t *>(at.data());
    std::vector<char> seen((size_t)p.nnz, 0);
    int64_t steps = 0, groups = 0;
    int32_t slice = 0;
    for (size_t c = 0; c + 1 < b.chunks.size(); ++c) {
        const SliceChunk &k = b.chunks[c];
        REQUIRE(k.nsteps >= 1 && k.nsteps * wide <= 256 && k.nsteps <= 64 && k.nleaves >= 1 && k.nleaves <= 256);
        REQUIRE(k.step0 == steps && k.group0 == groups && k.slice0 == slice);
        if (cap) REQUIRE(k.nsteps <= cap || cap < std::max(8, 64 / wide));
        int32_t group = 0;
        std::vector<int32_t> child(wide, -1);
        for (int32_t s = 0; s < k.nsteps; ++s) {
            REQUIRE(group < k.ngroups);
            for (int q = 0; q < wide; ++q) {
                const size_t o = (size_t)(steps + s) * wide + q;
                if (leaf[o] == 0xffffffffu) {
                    REQUIRE(place[o] == 255 && k.nleaves < 256);
                    continue;
                }
                REQUIRE(place[o] < k.nleaves);
                const int32_t z = k.leaf0 + place[o], f = t.fiber_of[z];
                REQUIRE(!seen[z]++ && (uint32_t)t.crd[2][z] == leaf[o] && t.slice_of[f] == slice);
                REQUIRE(gj[(size_t)(groups + group) * wide + q] == t.crd[1][f]);
                REQUIRE(child[q] < 0 || child[q] == f);
                child[q] = f;
            }
            if (k.gend >> s & 1) {
                std::fill(child.begin(), child.end(), -1);
                ++group;
            }
            if (k.send >> s & 1) {
                REQUIRE(k.gend >> s & 1);
                ++slice;
            }
        }
        REQUIRE(group == k.ngroups);
        steps += k.nsteps;
        groups += group;
    }
    for (char x : seen) REQUIRE(x == 1);
    REQUIRE(slice == t.nfib[0] && (size_t)groups * wide == gj.size());
    for (size_t r = 0; r + 1 < b.runs.size(); ++r) {
        const SliceRun &x = b.runs[r], &y = b.runs[r + 1];
        REQUIRE(x.step % 8 == 0 && x.step < b.chunks[x.chunk0].nsteps);
        REQUIRE(y.chunk0 > x.chunk0 || (y.chunk0 == x.chunk0 && y.step > x.step));
    }
    return 0;
}

int main()
{
    std::mt19937 rng(1);
    std::vector<std::vector<std::vector<int>>> shapes = {
        std::vector<std::vector<int>>(400, std::vector<int>(10, 20)), std::vector<std::vector<int>>(150, std::vector<int>(16, 16)),
        std::vector<std::vector<int>>(20, std::vector<int>(150, 13)), {{1}, {700}, {1}}, {{9}, {8}, {7}, {16}, {17}, {40}}};
    for (int n = 0; n < 40; ++n) {
        shapes.emplace_back(1 + rng() % (n % 5 ? 12 : 200));
        for (auto &slice : shapes.back()) {
            slice.resize(1 + rng() % (rng() % 9 ? 40 : 300));
            for (int &len : slice) len = n % 3 == 0 ? 9 + (int)(rng() % 32) : rng() % 3 ? 1 : 1 + (int)(rng() % (rng() % 30 ? 30 : 600));
        }
    }
    for (size_t n = 0; n < shapes.size(); ++n) {
        const Tensor t(shapes[n], rng);
        for (int tune : {0, 32})
            for (int cap : {0, 8, 16, 32, 64}) {
                auto one = [&](SliceSource src, int R, sc_dtype dtype, int piece) {
                    const int line = check(t, src, R, dtype, piece, cap, tune);
                    if (!line) return;
                    printf("shape %zu (%lld leaves), source %d, rank %d, pieces of %d, chunks of %d, runs %d: line %d\n", n, (long long)t.nfib[2], (int)src, R, piece, cap, tune, line);
                    exit(1);
                };
                for (int piece : {1, kSlicePiece}) one(SLICE_LEAVES, 16, SC_F32, piece);
                for (int piece : {kMttkrpPiece, kSlicePiece}) {
                    one(SLICE_MTTKRP, 16, SC_F32, piece);
                    one(SLICE_MTTKRP, 32, SC_F32, piece);
                    one(SLICE_MTTKRP, 16, SC_F64, piece);
                }
            }
    }
    return 0;
}
