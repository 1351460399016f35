#include "ewf_gen.h"

namespace ewf {

// =========================================================================================
// Col, held: chained reductions down short columns, and what is computed per element from them
//
// A workgroup of 1024 threads takes a strip of whole columns and holds it in registers: one read of the
// tensor, every level of the chain over the registers, one write, one launch, where a plan in passes takes three
// launches and reads the tensor twice (normalisation over a batch: the statistics, their fold, the normalised
// tensor).  TX lanes lie along the columns, 1024 / TX along the rows, NV rows to a thread.  A level's sums fold across
// the lanes of a wavefront, then every thread adds up the wavefronts' results of its own columns from LDS.

ewf_status Gen::gen_held()
{
    if (R != 2 || !c.reduced[0] || c.reduced[1]) return fail("held columns need one reduced dimension outside one kept dimension");
    const int64_t rows = c.extent[0], cols = c.extent[1];
    const int nin = g.ninputs, D = red.max_depth;
    if (!red.cross_nodes.empty()) return fail("held columns do not meet");
    // (beyond, strips that fit the registers are parts of lines: see below)
    if (rows > 4096) return fail("columns too long to be held");
    std::vector<int> ew_out_ops, group_out_ops;
    for (size_t k = nin; k < c.ops.size(); k++) {
        const bool group = (g.nodes[g.outputs[c.ops[k].index].value].bcast & red.axes) == red.axes;
        (group ? group_out_ops : ew_out_ops).push_back((int)k);
    }
    std::vector<std::vector<int>> lvl(D + 1);
    std::vector<int> early, late;
    for (int n : red.level_nodes) {
        const int op = g.nodes[n].op;
        // (every thread merges all wavefronts' results: cheap merges only)
        if (op == EWF_RARGMAX || op == kRSumSqCentred || op == kRSumExpShifted) return fail("held columns: a merge is too dear");
        lvl[red.edepth[n]].push_back(n);
        early.push_back(g.nodes[n].args[0]);
    }
    for (int k : ew_out_ops) late.push_back(g.outputs[c.ops[k].index].value);
    for (int k : group_out_ops) late.push_back(g.outputs[c.ops[k].index].value);
    // operands that vary along the rows: held where a reduction reads them, otherwise read for the outputs;
    // operands that do not: read once
    std::vector<int> held_ops, late_ops, col_ops;
    for (int k : inputs_of(needed(early))) (c.ops[k].stride[0] != 0 ? held_ops : col_ops).push_back(k);
    for (int k : inputs_of(needed(late))) {
        std::vector<int> &to = c.ops[k].stride[0] != 0 ? late_ops : col_ops;
        if (std::find(held_ops.begin(), held_ops.end(), k) == held_ops.end() && std::find(to.begin(), to.end(), k) == to.end()) to.push_back(k);
    }
    if (held_ops.empty()) return fail("nothing to hold");
    // (two columns a thread: a thread's folds cost by the column.  Batch normalisation of float16 [1024, 64] in
    // vectors of 2 / 4 / 8 3.8 / 4.7 / 7.5 us, float32 4.2 / 4.7; [2000, 4096] in 2 / 4 14.0 / 14.2)
    VEC = std::min(c.vec_loose, 2);
    const bool wide = c.vec < VEC;                          // vectors that assume element alignment only
    if (cols < VEC) return fail("fewer columns than a vector");
    int held_bytes = 0, moved = 0, narrowest = 4;
    auto rowwise = [&](int k) { return c.ops[k].stride[0] != 0 && c.ops[k].stride[1] == 1; };
    for (int k : held_ops) { if (!rowwise(k)) return fail("held columns: an operand without unit stride"); held_bytes += isz(c.ops[k].storage); }
    for (int k : late_ops) { if (!rowwise(k)) return fail("held columns: an operand without unit stride"); moved += isz(c.ops[k].storage); }
    for (int k : ew_out_ops) { if (!rowwise(k)) return fail("held columns: an output without unit stride"); moved += isz(c.ops[k].storage); narrowest = std::min(narrowest, isz(c.ops[k].storage)); }
    for (int k : held_ops) narrowest = std::min(narrowest, isz(c.ops[k].storage));
    moved += held_bytes;

    // ---- strips
    // What a strip width costs, in us: what the workgroups move, by the bytes of a row that a strip takes (parts of a
    // line are moved whole), or what a compute unit evaluates, 0.14 ns an element with eight operations.  Batch
    // normalisation, strips of 32 / 16 / 8 columns: float32 [2000, 4096] 14.0 / 16.4 / 41.2, [1200, 722] 8.1 / 7.2 / 7.6;
    // float16 [2000, 4000] 12.2 / 17.0 / 30.6, [1024, 4096] 8.0 / 10.6 / 21.7, [4096, 1024] 16.5 / 15.9 / 20.6, [3460, 116]
    // 10.0 / 7.9 / 7.4.  The plan in passes, its three kernels: 30.2, 10.5; 24.2, 20, 21.4, 10.7.  It stays where a strip
    // would be too narrow or too long: float32 [5000, 300] 14.0 in passes, 15.7 here; float16 [5000, 1001] 16.9 and 19.6, [5000, 300] 12.1 and 15.3.
    int operations = 0;
    for (size_t n = 0; n < g.nodes.size(); n++) operations += live[n] && g.nodes[n].kind == NodeKind::Apply;
    const int block = 1024, NW = block / 64;
    int TX = 0;
    double best = 0.95 * (10.0 + (double)c.total * (moved + held_bytes) / (narrowest == 2 ? 3.4e6 : 5.5e6));
    for (int tx = 1; tx <= 32; tx *= 2) {
        const int64_t w = (int64_t)tx * VEC, nv = ceil_div(rows, block / tx), strips = ceil_div(cols, w);
        if (tx > 1 && cols <= w / 2) break;
        if (nv * VEC * held_bytes > 64 * 4) continue;                          // 64 registers a thread
        const int64_t bytes = w * narrowest;
        if (bytes < 16 && cols > w) continue;
        const double share = (bytes >= 128 ? 1.0 : bytes >= 64 ? 0.8 : bytes >= 32 ? 0.2 : 0.1) * (wide ? 0.7 : 1.0);
        const double memory = (double)c.total * moved / 6.7e6 / share;
        const double arithmetic = (double)(rows * w) * 1.4e-4 * std::max(1.0, operations / 8.0) * std::max(1.0, (double)strips / device_cu_count());
        const double us = 3.8 + std::max(memory, arithmetic);
        if (us < best) { TX = tx; best = us; }
    }
    if (TX == 0) return fail("columns are better taken in passes");
    const int64_t W = std::min<int64_t>((int64_t)TX * VEC, cols), TY = block / TX, NV = ceil_div(rows, TY), NFULL = rows / TY;
    const int64_t strips = ceil_div(cols, W);
    const bool cut = cols % VEC != 0;
    // (Two threads, in two workgroups where the last strip is one column wide, own the columns that a cut vector shares: a
    // value that one of them may still read must stay.  Whole vectors are each workgroup's own, and its threads have read
    // what a column has one of before the first barrier.)
    for (size_t k = nin; cut && k < c.ops.size(); k++)
        if (c.ops[k].alias_of >= 0) return fail("held columns: a result in the place of an operand");
    p.block = block;
    p.tile[0] = rows;
    p.tile[1] = W;

    emit_header(block);
    build_layout();
    for (int l = 1; l <= D; l++) if (!lvl[l].empty()) emit_acc_struct("Acc" + std::to_string(l), lvl[l]);
    o << "extern \"C\" __global__ void __launch_bounds__(EWF_BLOCK) " << occupancy_attr() << "ewf_kernel(const Params p)\n{\n";
    o << "    const int tid = threadIdx.x, tx = tid & " << TX - 1 << ", ty = tid / " << TX << ";\n";
    int lds = 0;
    for (int l = 1; l <= D; l++) {
        if (lvl[l].empty()) continue;
        o << "    __shared__ Acc" << l << " sm" << l << "_[" << NW * TX * VEC << "];\n";
        lds += (int)(NW * TX * VEC * acc_bytes(lvl[l]));
    }
    if (lds > 60 * 1024) return fail("too many reductions for held columns (LDS)");
    // The vector that the last column cuts is read as the last whole one, also where that begins in the strip
    // before; the threads that share its columns compute and write the same values.
    o << "    const idx_t o0 = 0, o1 = (idx_t)blockIdx.x * " << W << " < p.ext[1] - EWF_VEC ? (idx_t)blockIdx.x * " << W << " : p.ext[1] - EWF_VEC;\n    (void)o0;\n";
    o << "    const int width_ = (int)((p.ext[1] - o1) < " << W << " ? (p.ext[1] - o1) : " << W << ");\n";
    o << "    const bool on_ = tx * EWF_VEC < width_;\n";
    o << "    const int at_ = tx * EWF_VEC < width_ - EWF_VEC ? tx * EWF_VEC : width_ - EWF_VEC;\n";
    const std::vector<int> dims = {0, 1};
    for (int k : held_ops) emit_base(k, dims, "    ");
    for (int k : late_ops) emit_base(k, dims, "    ");
    for (int k : col_ops) emit_base(k, dims, "    ");
    for (size_t k = nin; k < c.ops.size(); k++) emit_base((int)k, dims, "    ");
    auto at = [&](int k, const std::string &row) { return "ewf_at(q_" + opname(k) + ", (ioff_t)" + row + " * (ioff_t)p.st_" + opname(k) + "[0] + (ioff_t)at_)"; };
    auto load = [&](int k, const std::string &row) { return std::string(wide ? "ewf_ld_u<" : "ewf_ld<") + ctype(c.ops[k].storage) + ", EWF_VEC>(" + at(k, row) + ")"; };
    const std::string steps = "    #pragma unroll\n    for (int u = 0; u < " + std::to_string(NV) + "; ++u) {\n        const int r_ = ty + u * " + std::to_string(TY) + ";\n        (void)r_;\n";
    const std::string last_row = std::to_string(rows - 1);
    const std::string row_in = NFULL < NV ? "(u < " + std::to_string(NFULL) + " || r_ <= " + last_row + " ? r_ : " + last_row + ")" : std::string("r_");
    for (int k : held_ops) o << "    ewf_vec<" << ctype(c.ops[k].storage) << ", EWF_VEC> x_" << opname(k) << "[" << NV << "];\n";
    o << steps;
    for (int k : held_ops) o << "        x_" << opname(k) << "[u] = " << load(k, row_in) << ";\n";
    o << "    }\n";
    for (int k : col_ops) {
        o << "    " << ctype(c.ops[k].storage) << " h_" << opname(k) << "[EWF_VEC];\n";
        o << "    _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) h_" << opname(k) << "[e_] = q_" << opname(k) << "[(idx_t)(at_ + e_) * p.st_" << opname(k) << "[1]];\n";
    }
    EmitCtx cx;
    cx.input = [&](int k) {
        if (c.ops[k].stride[0] == 0) return "ewf_in(h_" + opname(k) + "[e_])";
        const std::string x = std::find(held_ops.begin(), held_ops.end(), k) != held_ops.end() ? "x_" + opname(k) + "[u]" : "l_" + opname(k);
        return c.ops[k].storage == EWF_F16 && VEC >= 2 ? "ewf_in_h(" + x + ", e_)" : "ewf_in(" + x + ".e[e_])";
    };
    cx.coord = [&](int d) { return d == 0 ? std::string("r_") : std::string("(o1 + at_ + e_)"); };
    auto results = [&](int below, const std::string &ind) {
        for (int l = 1; l < below; l++) if (!lvl[l].empty()) emit_results("acc" + std::to_string(l) + "[e_]", lvl[l], ind);
    };
    const std::string each = "_Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) ";
    for (int l = 1; l <= D; l++) {
        if (lvl[l].empty()) continue;
        const std::string an = "Acc" + std::to_string(l), av = "acc" + std::to_string(l), sm = "sm" + std::to_string(l) + "_";
        std::vector<int> tg;
        for (int n : lvl[l]) tg.push_back(g.nodes[n].args[0]);
        // (four chains of a thread's rows, met in pairs: in one chain of 32 the mean over 4096 float32 rows is off by
        // 4.5e-8, in passes 4.3e-8)
        const int chains = NV >= 8 ? 4 : 1;
        o << "    " << an << " sub" << l << "_[" << chains << "][EWF_VEC], " << av << "[EWF_VEC];\n";
        o << "    _Pragma(\"unroll\") for (int i_ = 0; i_ < " << chains << "; ++i_) " << each << "sub" << l << "_[i_][e_] = " << an << "_identity();\n";
        o << steps;
        if (NFULL < NV) o << "        if (u >= " << NFULL << " && r_ > " << last_row << ") continue;\n";
        o << "        " << each << "{\n";
        results(l, "            ");
        emit_values(needed(tg), cx, "            ");
        emit_accumulate("sub" + std::to_string(l) + "_[u & " + std::to_string(chains - 1) + "][e_]", lvl[l], [&](int node) { return argmax_index(node, cx.coord); }, "            ");
        o << "        }\n    }\n";
        const std::string sub = "sub" + std::to_string(l) + "_";
        if (chains == 1) o << "    " << each << av << "[e_] = " << sub << "[0][e_];\n";
        else o << "    " << each << av << "[e_] = " << an << "_combine()(" << an << "_combine()(" << sub << "[0][e_], " << sub << "[1][e_]), " << an << "_combine()(" << sub << "[2][e_], " << sub << "[3][e_]));\n";
        for (int m = TX; m < 64; m *= 2) o << "    " << each << av << "[e_] = " << an << "_combine()(" << av << "[e_], ewf_lane_xor(" << av << "[e_], " << m << "));\n";
        o << "    if ((tid & 63) < " << TX << ") { " << each << sm << "[((tid >> 6) * " << TX << " + tx) * EWF_VEC + e_] = " << av << "[e_]; }\n";
        o << "    __syncthreads();\n";
        // Four chains of four, which meet in pairs.  (All sixteen read at once took 16 registers a column.)
        o << "    {\n        " << an << " w_[4][EWF_VEC];\n";
        o << "        _Pragma(\"unroll\") for (int i_ = 0; i_ < 4; ++i_) " << each << "w_[i_][e_] = " << sm << "[(i_ * " << TX << " + tx) * EWF_VEC + e_];\n";
        o << "        _Pragma(\"unroll 1\") for (int j_ = 4; j_ < " << NW << "; j_ += 4)\n";
        o << "            _Pragma(\"unroll\") for (int i_ = 0; i_ < 4; ++i_) " << each << "w_[i_][e_] = " << an << "_combine()(w_[i_][e_], " << sm << "[((i_ + j_) * " << TX << " + tx) * EWF_VEC + e_]);\n";
        o << "        " << each << av << "[e_] = " << an << "_combine()(" << an << "_combine()(w_[0][e_], w_[1][e_]), " << an << "_combine()(w_[2][e_], w_[3][e_]));\n    }\n";
        // (every level starts from the operands alone: what one computed from them would be kept for the next)
        o << "    _Pragma(\"unroll\") for (int u = 0; u < " << NV << "; ++u) {";
        for (int k : held_ops) o << " ewf_forget(x_" << opname(k) << "[u]);";
        o << " }\n";
    }
    auto stored = [&](int k) { return std::string(c.ops[k].storage == EWF_F16 ? "ewf_out_f16" : c.ops[k].storage == EWF_I32 ? "ewf_out_i32" : "ewf_out_f32") + "(v" + std::to_string(g.outputs[c.ops[k].index].value) + ")"; };
    if (!ew_out_ops.empty()) {
        std::vector<int> tg;
        for (int k : ew_out_ops) tg.push_back(g.outputs[c.ops[k].index].value);
        o << "    if (on_) {\n" << steps;
        if (NFULL < NV) o << "        if (u >= " << NFULL << " && r_ > " << last_row << ") continue;\n";
        for (int k : late_ops) o << "        const ewf_vec<" << ctype(c.ops[k].storage) << ", EWF_VEC> l_" << opname(k) << " = " << load(k, "r_") << ";\n";
        for (int k : ew_out_ops) o << "        ewf_vec<" << ctype(c.ops[k].storage) << ", EWF_VEC> y_" << opname(k) << ";\n";
        o << "        " << each << "{\n";
        results(D + 1, "            ");
        emit_values(needed(tg), cx, "            ");
        for (int k : ew_out_ops) o << "            y_" << opname(k) << ".e[e_] = " << stored(k) << ";\n";
        o << "        }\n";
        for (int k : ew_out_ops) o << "        " << (wide ? "ewf_st_u<" : "ewf_st<") << ctype(c.ops[k].storage) << ", EWF_VEC>(" << at(k, "r_") << ", y_" << opname(k) << ");\n";
        o << "    }\n    }\n";
    }
    if (!group_out_ops.empty()) {
        std::vector<int> tg;
        for (int k : group_out_ops) tg.push_back(g.outputs[c.ops[k].index].value);
        o << "    if (tid < " << TX << " && on_) {\n        " << each << "{\n";
        results(D + 1, "            ");
        emit_values(needed(tg), cx, "            ");
        for (int k : group_out_ops) o << "            q_" << opname(k) << "[(idx_t)(at_ + e_) * p.st_" << opname(k) << "[1]] = " << stored(k) << ";\n";
        o << "        }\n    }\n";
    }
    o << "}\n";

    // ---- launch geometry and argument block
    p.grid = strips;
    p.lds_bytes = lds;
    p.staged = 0;
    p.workspace_bytes = 0;
    p.finish_grid = 0;
    p.args.assign(p.layout.size, 0);
    auto put_idx = [&](const std::string &name, int i, int64_t v) {
        int f = p.layout.find(name);
        size_t off = p.layout.offsets[f];
        if (c.idx64) memcpy(&p.args[off + 8 * (size_t)i], &v, 8);
        else { int32_t w = (int32_t)v; memcpy(&p.args[off + 4 * (size_t)i], &w, 4); }
    };
    for (int d = 0; d < R; d++) put_idx("ext", d, c.extent[d]);
    put_idx("ntile", 0, 1);
    put_idx("ntile", 1, strips);
    put_idx("ntiles", 0, strips);
    put_idx("nrows", 0, cols);
    put_idx("nslots", 0, 1);
    for (size_t k = 0; k < c.ops.size(); k++)
        for (int d = 0; d < R; d++) put_idx("st_" + opname((int)k), d, c.ops[k].stride[d]);
    p.source = o.str();
    return EWF_OK;
}

}  // namespace ewf
