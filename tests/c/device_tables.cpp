// Writes the tables the kernels read of a mechanism to standard output, each
// as "name type count\n" and the raw values: device_tables <mechanism> <lanes>.
// Host sources only; built with the standard library's bounds checks.
#include <cstdio>
#include <fstream>
#include <iostream>
#include <sstream>

#include "mech.hpp"

static void put(const char *name, const char *type, const void *p, size_t count, size_t size)
{
    std::printf("%s %s %zu\n", name, type, count);
    std::fwrite(p, size, count, stdout);
}
static void put(const std::string &name, const std::vector<uint16_t> &v) { put(name.c_str(), "uint16", v.data(), v.size(), 2); }
static void put(const std::string &name, const std::vector<uint32_t> &v) { put(name.c_str(), "uint32", v.data(), v.size(), 4); }
static void put(const std::string &name, const std::vector<int> &v) { put(name.c_str(), "int32", v.data(), v.size(), 4); }
static void put(const std::string &name, const std::vector<double> &v) { put(name.c_str(), "float64", v.data(), v.size(), 8); }

static void put(const std::string &name, const sc::SparseRx &x)
{
    put(name + ".counts", std::vector<int>{x.passes, x.n_tb, x.n_troe});
    put(name + ".order", x.order);
    put(name + ".rec", x.rec);
    put(name + ".ix", x.ix);
    put(name + ".ixe", x.ixe);
    put(name + ".eam1", x.eam1);
    put(name + ".troe", x.troe);
}

int main(int argc, char **argv)
{
    if (argc != 3) return 2;
    std::ifstream f(argv[1]);
    std::stringstream text;
    text << f.rdbuf();
    const int lanes = std::atoi(argv[2]);
    try {
        const sc::Mech m = sc::load_mechanism(text.str());
        const sc::SparseDev d = sc::sparse_device(m, lanes);
        put("size", std::vector<int>{m.N, m.R, m.sp.n, m.sp.nnz, m.n_padded});
        put("region", std::vector<int>{sc::sparse_region(m.sp.n, m.sp.nnz, lanes), sc::SPL_E});
        // waves a workgroup by the regions a CU of 160 KB holds, up to two waves
        // per SIMD with one slot per lane, one with two: for 64 to 2^20 cells
        const int vpl = m.sp.n <= 64 ? 1 : 2;
        int groups[sc::CREW_SIZES] = {};
        for (int k = 0; k < (vpl == 1 ? 3 : 2); ++k) {
            const int bytes = 128 + 8 * sc::sparse_region(m.sp.n, m.sp.nnz, 64) * (vpl == 1 ? 1 << k : 1);
            groups[k] = 256 * std::min(sc::lds_held(bytes), (vpl == 1 ? 8 : 4) >> k);
        }
        std::vector<int> crews(groups, groups + sc::CREW_SIZES);
        for (int64_t n = 64; n <= 1 << 20; n *= 2) crews.push_back(sc::crew_choice(vpl, groups, 1 << 30, n));
        put("crews", crews);
        std::vector<int> leaves;
        for (int vpl : {1, 2})
            for (int waves : {1, 2, 4})
                for (int w : {1, waves}) leaves.insert(leaves.end(), {vpl, w, waves, sc::crew_leaves(vpl, w, waves)});
        put("leaves", leaves);
        put("pos", m.sp.pos);
        put("erow", m.sp.erow);
        put("ecol", m.sp.ecol);
        put("row", d.row);
        put("low", d.low);
        put("up", d.up);
        put("blk", d.blk);
        put("comp", d.comp);
        put("sparse", sc::sparse_reactions(m, lanes));
        if (m.N + 1 <= sc::MAX_STATE) put("dense", sc::dense_reactions(m));
    } catch (const std::exception &e) {
        std::cerr << e.what() << "\n";
        return 1;
    }
    return 0;
}
