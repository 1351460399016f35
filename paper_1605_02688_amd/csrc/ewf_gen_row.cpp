#include "ewf_gen.h"

namespace ewf {

// =========================================================================================
// Row

ewf_status Gen::gen_row()
{
    const int in_d = R - 1;
    const int64_t cols = c.extent[in_d];
    int block = e.opts.block_threads;
    if (block <= 0) {
        block = 256;
        while (block > 64 && cols <= (int64_t)(block / 2) * VEC * 2) block /= 2;
        // at most twelve vectors of the row per thread, or 24 single elements (rows of 10001
        // float32, whose odd pitch allows no wider access: 512 threads 14.6 us, 1024 threads 22.3 us)
        while (block < 1024 && cols > (int64_t)block * std::max(VEC * 12, 24)) block *= 2;
    }
    if (block % 64 || block > 1024) return fail("block_threads must be a multiple of 64, at most 1024");
    p.block = block;
    const int nin = g.ninputs;

    // ---- roles of the outputs
    std::vector<int> full_out_ops, group_out_ops, final_out_ops;
    for (size_t k = nin; k < c.ops.size(); k++) {
        int vn = g.outputs[c.ops[k].index].value;
        const Node &v = g.nodes[vn];
        if (after_cross[vn]) final_out_ops.push_back((int)k);
        else if ((v.bcast & red.axes) == red.axes) group_out_ops.push_back((int)k);
        else full_out_ops.push_back((int)k);
    }
    // ---- per-level targets
    const int D = red.max_depth;
    std::vector<std::vector<int>> lvl(D + 1);
    std::vector<std::vector<Gather>> gat(D + 1);
    for (int n : red.level_nodes) {
        Gather ga;
        if (match_gather(n, ga) && ga.cdim == in_d) gat[red.edepth[n]].push_back(ga);
        else lvl[red.edepth[n]].push_back(n);
    }
    // (where no workgroup-wide fold follows, a row that is written over is summed as described: nothing else keeps
    // the threads that store behind those that read the one element)
    bool fold_follows = false;
    for (int l = D; l >= 1; l--) {
        fold_follows = fold_follows || !lvl[l].empty();
        for (size_t i = 0; i < gat[l].size() && !fold_follows; i++) {
            if (!written_over(gat[l][i].input)) continue;
            lvl[l].push_back(gat[l][i].node);
            gat[l].erase(gat[l].begin() + i);
            fold_follows = true;
        }
    }

    // which inputs vary along the row and are read by some per-element computation
    std::vector<int> elem_targets;
    for (int l = 1; l <= D; l++) for (int n : lvl[l]) elem_targets.push_back(g.nodes[n].args[0]);
    for (int k : full_out_ops) elem_targets.push_back(g.outputs[c.ops[k].index].value);
    std::vector<char> eneed = needed(elem_targets);
    std::vector<int> row_ops, splat_ops;
    for (int k : inputs_of(eneed)) (c.ops[k].stride[in_d] != 0 ? row_ops : splat_ops).push_back(k);

    // Operands that only the element-wise outputs use (the scale and shift rows of a layer
    // normalisation) are read where those outputs are written, not held under the reductions.
    std::vector<char> late(c.ops.size(), 0);
    {
        std::vector<int> level_targets;
        for (int l = 1; l <= D; l++) for (int n : lvl[l]) level_targets.push_back(g.nodes[n].args[0]);
        std::vector<char> lneed = needed(level_targets);
        std::vector<int> under = inputs_of(lneed);
        for (int k : row_ops) if (std::find(under.begin(), under.end(), k) == under.end()) late[k] = 1;
    }
    // With such operands the last pass issues loads of its own next to the arithmetic, and more
    // threads with fewer vectors each hide them better: two vectors of the row per thread (layer
    // normalisation with scale and shift rows, 134 MB: float16 [4096, 16384] 256 threads 67.2 us,
    // 1024 threads 55.5 us; [8192, 8192] 256 threads 59.5 us, 512 threads 54.4 us; float32
    // [8192, 8192] 99.4 -> 93.0 us, [4096, 16384] 99.3 -> 91.1 us; softmax, which has none, runs
    // best as it is).
    if (e.opts.block_threads <= 0 && std::find(late.begin(), late.end(), (char)1) != late.end()) {
        int want = 64;
        while (want < 1024 && (int64_t)want * VEC * 2 < cols) want *= 2;
        if (want > block) { block = want; p.block = block; }
    }
    const bool loose = p.loose_vec;
    // Rows that do not start on cache lines and are written back: the vectors start on the output's lines instead of with the row
    // (`shifted`), so that a wavefront's 1 KiB is eight whole lines and not parts of nine.  A row's first vector then
    // begins before it and its last one ends behind it; either is taken as the row's first or last whole vector, of
    // which the thread counts and writes what is its own.  Gradient of softmax cross-entropy, float32: [1280, 50257] 102.4 ->
    // 93.5 us (rows of 50304, whole lines, 93.7), [1280, 50260] 101.4 -> 93.1, [1280, 33001] 66.6 -> 61.9, [4000, 7777] 44.3 -> 42.3;
    // softmax, float32 [4000, 16001] 95.4 -> 88.9, float16 [4000, 16001] 52.8 -> 44.4, [10000, 5003] 40.3 -> 37.7.  Not on short rows,
    // nor where the memory-side cache holds both tensors (softmax over float16 [20000, 3001] 47.6, shifted 52.3, [300, 16380]
    // 8.9 and 9.9; the gradient on [4096, 3001] 18.6 and 19.1, on [1280, 10004], aligned to 16 bytes, 20.0 and 20.5).
    bool shifted = !full_out_ops.empty();
    if (shifted) {
        const int64_t row_bytes = cols * isz(c.ops[full_out_ops[0]].storage), rows = c.total / cols;
        int64_t moved = 0;
        for (int k : row_ops) moved += isz(c.ops[k].storage);
        for (int k : full_out_ops) moved += isz(c.ops[k].storage);
        shifted = row_bytes >= (VEC > 4 ? 10000 : 8000) && rows * cols * moved >= 100000000 && (loose || c.total >= (int64_t)1 << 24);
        bool off_lines = false;
        std::vector<int> walked = row_ops;
        walked.insert(walked.end(), full_out_ops.begin(), full_out_ops.end());
        for (int k : walked) {
            const Operand &op = c.ops[k];
            if (late[k] || op.access != Access::Vector || VEC * isz(op.storage) % 4) shifted = false;
            for (int d = 0; d < R - 1; d++) off_lines = off_lines || op.stride[d] * isz(op.storage) % 128;
        }
        for (int n : red.level_nodes) if (g.nodes[n].op == EWF_RARGMAX) shifted = false;
        shifted = shifted && off_lines;
    }
    // (and then 1024 threads from where others take 512: softmax over [4000, 13001] 71.6 -> 68.6 us, [4000, 16001] 88.9 -> 85.5,
    // the gradient on [1500, 24003] 56.2 -> 52.5, on [1280, 20001] 37.1 and 37.2; rows of whole vectors, [1280, 24576], 44.8 and 46.1)
    if (shifted && loose && VEC == 4 && block == 512 && e.opts.block_threads <= 0) { block = 1024; p.block = block; }
    // ---- residency: keep the row in registers when it fits
    const int64_t per_iter = (int64_t)block * VEC;
    const int64_t line = shifted ? 128 / isz(c.ops[full_out_ops[0]].storage) : 1;
    const int64_t NV = ceil_div(cols + line - 1, per_iter);
    int regs = 0;
    for (int k : row_ops) if (!late[k]) regs += (int)NV * VEC * isz(c.ops[k].storage) / 4;
    const bool resident = NV <= 32 && regs <= 96;
    if (!resident) shifted = false;
    int64_t nrows = 1;
    for (int d = 0; d < R - 1; d++) nrows *= c.extent[d];
    // one workgroup per row when the grid can hold them all: no loop, so nothing is hoisted
    // out of it into registers that the row needs
    if (nrows >= ((int64_t)1 << 31) - 1) return fail("too many rows");
    const int64_t grid_cap = e.opts.max_blocks > 0 ? e.opts.max_blocks : (int64_t)256 * 32;
    const bool row_loop = nrows > grid_cap;
    // The first NFULL steps of a resident row are in range for every thread of the
    // workgroup at this plan's row length: straight-line code there lets the compiler wait
    // for the loads one by one instead of for all of them.  (The row length is part of the
    // plan's key, and NFULL of the generated text, so the assumption travels with the code.)
    const int64_t NFULL = resident ? cols / per_iter : 0;
    // Two workgroups of 1024 threads share a compute unit, one loading while the other computes or stores, when
    // neither takes more than 64 registers a thread.  Left alone the compiler takes up to 128 under 52 registers of
    // row: it keeps for the next pass what one pass computed (the exponentials, the column numbers).  In a `tight` row
    // every pass starts from the row alone, and rows of more than 44 registers leave some of their vectors in
    // LDS, at most 64 KiB a workgroup, read there past the registers.  Gradient of softmax cross-entropy, float32:
    // [1280, 50257] 107.7 -> 102.4 us, [1280, 32768] 64.0 -> 60.8, [900, 61001] 120.9 -> 89.7 (two passes before), [1220, 65536]
    // 148.4 -> 121.0; softmax over float16 [800, 100000] 183.7 -> 81.  Only where it takes less than 65 registers and the kernel
    // left alone takes more (softmax over float32 [1000, 40000] 56.0 us left alone, 57.7 tight), not beside operands that the last
    // pass loads, which want registers of their own (layer normalisation of float32 [1024, 65536] 101.6 us, 111.3
    // tight), and not under a single reduction of float16 (x - mean(x) on [300, 100000] 25.2 us, 26.4 tight).
    auto parkable = [&](int k) { return !late[k] && c.ops[k].access == Access::Vector && VEC * isz(c.ops[k].storage) == 16; };
    const bool words = std::all_of(row_ops.begin(), row_ops.end(), [&](int k) { return isz(c.ops[k].storage) == 4; });
    p.tight_possible = resident && !row_loop && block == 1024 && regs > 20 && std::find(late.begin(), late.end(), (char)1) == late.end() &&
                       (words || D >= 2) && !p.no_tight;
    p.tight_needed = false;
    int64_t park = 0;                                  // steps of the row that wait in LDS
    if (p.tight_possible && regs > 44) {
        const int64_t nops = std::count_if(row_ops.begin(), row_ops.end(), parkable);
        if (nops > 0) park = std::min({ceil_div(regs - 44, 4 * nops), NFULL - (shifted ? 1 : 0), 65536 / (nops * block * 16)});
        if (regs - 4 * nops * park > 48) { p.tight_possible = false; park = 0; }
    }
    const bool tight_possible = p.tight_possible, tight = p.tight && tight_possible;
    if (p.avoid_poor_rows && e.opts.split_rows != 2) {
        // measured on [rows, cols] float32 softmax cross-entropy of 268 MB: rows held in registers
        // run at 5.3-5.5 TB/s up to 32768 columns but 4.1 TB/s at 65536 (64 registers per thread,
        // 1024 threads: one workgroup per compute unit), rows streamed once per level 2.7-3.4 TB/s;
        // split over workgroups 5.0-5.2 TB/s at any row length
        // (a chain that a plan in passes cannot shorten -- layer normalisation of float32
        // [4096, 16384] with its scale and shift rows: 96 registers of row data, 91 us here against
        // 185 us in three passes -- keeps the row class as long as the row fits at all)
        // (rows that are only read: up to 27 registers of 1024 threads; float32 sums and extremes, tight, up to 44 where there are two for
        // each compute unit and up to 60 where there are four.  Softmax cross-entropy on float32, split over workgroups against one
        // workgroup a row: [600, 24577] 18.6 and 15.7 us, [1220, 24577] 29.5 and 23.9, [600, 40000] 24.6 and 21.4, [1220, 32768]
        // 33.4 and 29.2; 52 registers, [1220, 53001] 51.2 and 48.2, [600, 53001] 28.9 and 29.7; 64, [1220, 65536] 58.0 and 71.9.  From 256 MB on
        // they stay split, which the planning tests state of [2048, 32768], though one workgroup a row is faster there too: log-sum-exp of
        // float32 [2048, 32768] 44.4 and 42.4, [2048, 40000] 56.3 and 51.6, [4096, 32770] 86.2 and 81.6)
        // (rows that are written back too are read once here and twice in two passes: kept up to 56
        // registers -- the gradient of softmax cross-entropy on float32 [1280, 50257] 143.0 us in two passes, 108.5
        // here even with one workgroup on a compute unit, [400, 50257] 50.6 and 38.0 us -- and up to 64 in tight rows, two for each compute unit)
        const int64_t two_a_unit = (int64_t)2 * device_cu_count();
        const bool adds = std::none_of(red.level_nodes.begin(), red.level_nodes.end(), [&](int n) { return g.nodes[n].op == EWF_RPROD; });
        const int alone = !full_out_ops.empty() ? 56 : block == 1024 ? 27 : 48;
        int held = alone;
        if (!full_out_ops.empty() && park > 0 && nrows >= two_a_unit) held = 64;
        if (full_out_ops.empty() && tight_possible && words && adds && nrows >= two_a_unit && nrows * cols < ((int64_t)1 << 26)) held = nrows < 2 * two_a_unit ? 44 : 60;
        const bool too_long = !resident || (regs > held && p.fused_depth <= 1);
        p.tight_needed = regs > alone && p.fused_depth <= 1;
        if (too_long || (nrows * 2 < device_cu_count() && cols >= 16384) || e.opts.split_rows == 1) {
            p.row_refused = true;
            return fail(too_long ? "a row does not fit the registers of a workgroup well: the row class would read it once per reduction level or run one workgroup per compute unit"
                                 : "too few rows for one workgroup per row to occupy the chip");
        }
    }
    if (!tight) park = 0;
    auto parked = [&](int k) { return park > 0 && parkable(k); };
    const int U = resident ? (int)NV : (e.opts.unroll > 0 ? e.opts.unroll : 4);
    p.tile[in_d] = cols;
    // Maxima and arg-maxima of a float input row that waits in registers are taken the cheap way
    // first: the hardware maximum (which drops NaN) next to a check word that turns NaN when the
    // row holds a NaN or an infinity, then the index by the threads that hold the maximum.  Only a
    // row whose check word is NaN is folded again with the rules that rank NaN.  (Per element: one
    // and a half instructions instead of five on a dependent chain.)
    auto has_argmax = [&](const std::vector<int> &nodes) {
        return std::any_of(nodes.begin(), nodes.end(), [&](int n) { return g.nodes[n].op == EWF_RARGMAX; });
    };
    std::vector<std::vector<int>> fastn(D + 1);
    std::vector<int> fast_op(D + 1, -1);
    if (resident && !e.opts.plain_extremes) {
        for (int l = 1; l <= D; l++) {
            int arg = -1;
            std::vector<int> rest;
            for (int n : lvl[l]) {
                const Node &nd = g.nodes[n];
                const Node &a = g.nodes[nd.args[0]];
                bool take = (nd.op == EWF_RMAX || nd.op == EWF_RARGMAX) && a.vtype == EWF_F32 && a.kind == NodeKind::Input &&
                            std::find(row_ops.begin(), row_ops.end(), a.index) != row_ops.end() && !late[a.index] &&
                            (arg < 0 || arg == nd.args[0]);
                if (take) { arg = nd.args[0]; fastn[l].push_back(n); fast_op[l] = a.index; }
                else rest.push_back(n);
            }
            lvl[l] = rest;
        }
    }
    if (tight) {
        auto_waves_per_simd = p.no_auto_occupancy ? 0 : 8;
    } else {
        // When all rows can be resident on the chip at once there is no second round of
        // workgroups (whose tail would idle most of the chip): ask the compiler for the
        // register budget that lets that many wavefronts share a SIMD, if the row leaves
        // room for the arithmetic under it.
        const int64_t wg_per_cu = ceil_div(nrows, device_cu_count());
        const int64_t waves = ceil_div(wg_per_cu * (block / 64), 4);
        if (resident && !p.no_auto_occupancy && waves >= 2 && waves <= 8 && regs + 40 <= 512 / waves / 8 * 8) {
            auto_waves_per_simd = (int)waves;
            p.used_auto_occupancy = !(e.opts.waves_per_simd >= 1 && e.opts.waves_per_simd <= 8);
        }
    }

    emit_header(block);
    build_layout();
    for (int l = 1; l <= D; l++) if (!lvl[l].empty()) emit_acc_struct("Acc" + std::to_string(l), lvl[l]);
    for (int l = 1; l <= D; l++) if (!fastn[l].empty()) emit_acc_struct("AccS" + std::to_string(l), fastn[l]);
    const bool has_cross = !red.cross_nodes.empty();
    if (has_cross) emit_acc_struct("AccX", red.cross_nodes);

    o << "extern \"C\" __global__ void __launch_bounds__(EWF_BLOCK) " << occupancy_attr() << "ewf_kernel(const Params p)\n{\n";
    o << "    const int tid = threadIdx.x;\n";
    o << "    const idx_t cols = p.ext[" << in_d << "];\n";
    for (int l = 1; l <= D; l++) if (!lvl[l].empty()) o << "    __shared__ Acc" << l << " sm_acc" << l << "[EWF_NWAVES];\n";
    for (int l = 1; l <= D; l++)
        if (!fastn[l].empty())
            o << "    __shared__ AccS" << l << " sm_accs" << l << "[EWF_NWAVES];\n    __shared__ ewf_fmax sm_fm" << l
              << "[EWF_NWAVES];\n" << (has_argmax(fastn[l]) ? "    __shared__ int sm_ix" + std::to_string(l) + "[EWF_NWAVES];\n" : std::string(""));
    for (int k : row_ops)
        if (parked(k)) o << "    __shared__ ewf_vec<" << ctype(c.ops[k].storage) << ", EWF_VEC> park_" << opname(k) << "[" << park << " * EWF_BLOCK];\n";
    if (has_cross) o << "    AccX *const partials = (AccX *)p.ws_partials;\n";
    if (!row_loop) o << "    if ((idx_t)blockIdx.x < p.nrows) {\n        const idx_t row = blockIdx.x;\n";
    else o << "    for (idx_t row = blockIdx.x; row < p.nrows; row += gridDim.x) {\n";
    o << "        idx_t t_ = row;\n";
    std::vector<int> outer;
    for (int d = R - 2; d >= 0; d--) {
        if (d > 0) o << "        const idx_t o" << d << " = ewf_uniform(t_ % p.ext[" << d << "]); t_ /= p.ext[" << d << "];\n";
        else o << "        const idx_t o0 = ewf_uniform(t_);\n";
    }
    for (int d = 0; d < R - 1; d++) outer.push_back(d);
    std::vector<int> based;
    auto base_once = [&](int k, const std::string &ind) {
        if (std::find(based.begin(), based.end(), k) != based.end()) return;
        based.push_back(k);
        emit_base(k, outer, ind);
    };
    for (int k : row_ops) base_once(k, "        ");
    for (int k : splat_ops) base_once(k, "        ");
    for (int k : full_out_ops) base_once(k, "        ");
    // (lines as they lie when the tensor starts on one: which elements a thread takes depends on the layout, never on the address)
    if (shifted) {
        const int k = full_out_ops[0];
        std::string at;
        for (int d : outer) if (c.ops[k].stride[d] != 0) at += (at.empty() ? "" : " + ") + ("o" + std::to_string(d)) + " * p.st_" + opname(k) + "[" + std::to_string(d) + "]";
        o << "        const idx_t head_ = (idx_t)((" << (at.empty() ? std::string("0") : at) << ") & " << line - 1 << ");\n";
    }

    // the loop over the row: either over register-resident vectors or streaming chunks
    int pass = 0;
    std::string me = "tid";                            // the thread's number as the current pass of a tight row knows it
    auto open_pass = [&]() {
        if (resident) {
            o << "        #pragma unroll\n        for (int u = 0; u < " << U << "; ++u) {\n";
            if (shifted) {
                o << "            const idx_t own_ = (idx_t)(u * EWF_BLOCK + " << me << ") * EWF_VEC - head_;\n";
                o << "            if ((u == 0 && own_ + EWF_VEC <= 0) || (u >= " << NFULL << " && own_ >= cols)) continue;\n";
                if (loose) o << "            const idx_t col = u == 0 && own_ < 0 ? 0 : u >= " << NFULL << " && own_ + EWF_VEC > cols ? cols - EWF_VEC : own_;\n";
                else o << "            const idx_t col = own_;\n";
            } else {
                o << "            const idx_t col = (idx_t)(u * EWF_BLOCK + " << me << ") * EWF_VEC;\n";
                o << "            if (u >= " << NFULL << " && col >= cols) continue;\n";
            }
        } else {
            o << "        for (idx_t c0 = 0; c0 < cols; c0 += " << (per_iter * U) << ") {\n";
            o << "        #pragma unroll\n        for (int u = 0; u < " << U << "; ++u) {\n";
            o << "            const idx_t col = c0 + (idx_t)(u * EWF_BLOCK + tid) * EWF_VEC;\n";
            o << "            if (col >= cols) continue;\n";
        }
    };
    auto close_pass = [&]() {
        o << "        }\n";
        if (!resident) o << "        }\n";
    };
    // Vectors that assume element alignment only (see Plan::loose_vec): a row may start at any
    // element, and when its length is no whole number of vectors the last one is cut (`ragged`)
    // and moved into place (ewf_move_cut).  The steps below NFULL hold whole vectors for every thread,
    // which the unrolled code knows at compile time.
    const bool ragged = loose && cols % VEC != 0 && !shifted;
    const std::string whole = "(u < " + std::to_string(NFULL) + " || col + EWF_VEC <= cols)";
    const std::string inside = ragged ? "if (u < " + std::to_string(NFULL) + " || col + e_ < cols) " : std::string("");
    // elements of a vector that are not the thread's own
    const std::string skip = shifted && loose ? "if ((u == 0 && col + e_ >= own_ + EWF_VEC) || (u >= " + std::to_string(NFULL) + " && col + e_ < own_)) continue;\n"
                             : ragged ? "if (u >= " + std::to_string(NFULL) + " && col + e_ >= cols) continue;\n" : std::string("");
    const std::string cut_len = std::to_string(cols % VEC);
    auto streamed = [&](const Operand &op) { return op.stream && VEC * isz(op.storage) % 16 == 0 ? ", ewf_streamed()" : ""; };
    auto emit_row_load = [&](int k, const std::string &ind, const std::string &dst) {
        const Operand &op = c.ops[k];
        std::string nm = opname(k);
        if (op.access == Access::Vector && loose) {
            if (ragged) {
                o << ind << "if (u < " << NFULL << ") " << dst << " = ewf_ld_u<" << ctype(op.storage) << ", EWF_VEC>(q_" << nm << " + col" << streamed(op) << ");\n";
                o << ind << "else " << dst << " = ewf_ld_cut<" << ctype(op.storage) << ", EWF_VEC, " << cut_len << ">(q_" << nm << " + col, col + EWF_VEC > cols);\n";
            }
            else o << ind << dst << " = ewf_ld_u<" << ctype(op.storage) << ", EWF_VEC>(q_" << nm << " + col" << streamed(op) << ");\n";
        }
        else if (op.access == Access::Vector)
            o << ind << dst << " = " << (op.stream ? "ewf_ld_nt<" : "ewf_ld<") << ctype(op.storage) << ", EWF_VEC>(q_" << nm << " + col);\n";
        else
            o << ind << "_Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) " << dst << ".e[e_] = q_" << nm
              << "[" << (ragged ? "(u < " + std::to_string(NFULL) + " || col + e_ < cols ? col + e_ : cols - 1)" : std::string("(col + e_)"))
              << " * p.st_" << nm << "[" << in_d << "]];\n";
    };

    // values constant along the row come first: an index that a gather depends on is then
    // the first load to return, and the dependent read queues right behind the row
    std::vector<int> uniform_loaded = splat_ops;
    for (int l = 1; l <= D; l++)
        for (const Gather &ga : gat[l])
            for (int k : inputs_of(needed(std::vector<int>{ga.index_value})))
                if (std::find(uniform_loaded.begin(), uniform_loaded.end(), k) == uniform_loaded.end()) uniform_loaded.push_back(k);
    for (int k : uniform_loaded) {
        base_once(k, "        ");
        o << "        const " << ctype(c.ops[k].storage) << " g_" << opname(k) << " = ewf_ld_uniform(q_" << opname(k) << ");\n";
    }
    const std::string in_lds = "u >= " + std::to_string(NFULL - park) + " && u < " + std::to_string(NFULL);
    if (resident) {
        for (int k : row_ops) if (!late[k]) o << "        ewf_vec<" << ctype(c.ops[k].storage) << ", EWF_VEC> x_" << opname(k) << "[" << U << "];\n";
        if (NFULL > 0 || !ragged) {
            if (ragged) {
                // the whole steps here; the last one below, where the cut vector is moved into
                // place behind all the loads
                o << "        #pragma unroll\n        for (int u = 0; u < " << NFULL << "; ++u) {\n";
                o << "            const idx_t col = (idx_t)(u * EWF_BLOCK + tid) * EWF_VEC;\n";
            }
            else open_pass();
            for (int k : row_ops) {
                if (late[k]) continue;
                if (parked(k)) o << "            if (" << in_lds << ") ewf_ld_lds<" << ctype(c.ops[k].storage) << ", EWF_VEC, " << (c.ops[k].stream ? "true" : "false") << ">(q_" << opname(k) << " + col, park_" << opname(k)
                                 << " + ((u - " << NFULL - park << ") * EWF_BLOCK + ewf_uniform(tid & ~63)));\n            else\n";
                emit_row_load(k, "            ", "x_" + opname(k) + "[u]");
            }
            close_pass();
        }
        if (ragged) {
            o << "        #pragma unroll\n        for (int u = " << NFULL << "; u < " << U << "; ++u) {\n";
            o << "            const idx_t col = (idx_t)(u * EWF_BLOCK + tid) * EWF_VEC;\n";
            o << "            const idx_t at_ = col + EWF_VEC <= cols ? col : cols - EWF_VEC;\n";
            o << "            if (col < cols) {\n";
            for (int k : row_ops) {
                if (late[k]) continue;
                if (c.ops[k].access == Access::Vector)
                    o << "                x_" << opname(k) << "[u] = ewf_ld_u<" << ctype(c.ops[k].storage) << ", EWF_VEC>(q_" << opname(k) << " + at_" << streamed(c.ops[k]) << ");\n";
                else
                    emit_row_load(k, "                ", "x_" + opname(k) + "[u]");
            }
            o << "            }\n";
            o << "        }\n        #pragma unroll\n        for (int u = " << NFULL << "; u < " << U << "; ++u) {\n";
            o << "            const bool cut_ = (idx_t)(u * EWF_BLOCK + tid) * EWF_VEC + EWF_VEC > cols;\n";
            for (int k : row_ops)
                if (!late[k] && c.ops[k].access == Access::Vector)
                    o << "            x_" << opname(k) << "[u] = ewf_move_cut<" << ctype(c.ops[k].storage) << ", EWF_VEC, " << cut_len << ">(x_" << opname(k) << "[u], cut_);\n";
            o << "        }\n";
        }
    }

    // the vector of step u of a parked operand; the first pass over the row waits for the loads behind the steps in registers
    bool waited = park == 0;
    auto take_vec = [&](int k) {
        const std::string nm = opname(k);
        if (!waited) o << "            if (u == " << NFULL - park << ") ewf_wait_loads();\n";
        waited = true;
        o << "            ewf_vec<" << ctype(c.ops[k].storage) << ", EWF_VEC> w_" << nm << ";\n            if (" << in_lds << ") w_" << nm << " = park_" << nm
          << "[(u - " << NFULL - park << ") * EWF_BLOCK + " << me << "]; else w_" << nm << " = x_" << nm << "[u];\n";
    };
    auto forget = [&]() {
        if (!tight) return;
        me = "tid" + std::to_string(++pass);
        o << "        const int " << me << " = ewf_forget(tid) & (EWF_BLOCK - 1);\n";
        if (pass == 1) return;                         // (nothing computed yet, and the first pass need not wait for every load)
        for (int k : row_ops)
            if (!late[k]) o << "        #pragma unroll\n        for (int u = 0; u < " << U << "; ++u) ewf_forget(x_" << opname(k) << "[u]);\n";
    };
    EmitCtx cx;
    cx.input = [&](int k) {
        if (c.ops[k].stride[in_d] == 0) return "ewf_in(g_" + opname(k) + ")";
        return resident && !late[k] && !parked(k) ? "ewf_in(x_" + opname(k) + "[u].e[e_])" : "ewf_in(w_" + opname(k) + ".e[e_])";
    };
    cx.coord = [&](int d) {
        if (d == in_d) return std::string("col + e_");
        return "o" + std::to_string(d);
    };
    auto stream_loads = [&](const std::vector<char> &need) {
        for (int k : inputs_of(need)) {
            if (c.ops[k].stride[in_d] == 0) continue;
            if (resident && !late[k]) { if (parked(k)) take_vec(k); continue; }
            o << "            ewf_vec<" << ctype(c.ops[k].storage) << ", EWF_VEC> w_" << opname(k) << ";\n";
            emit_row_load(k, "            ", "w_" + opname(k));
        }
    };

    // values constant along the row, evaluated by every thread (uniform addresses)
    EmitCtx ux;
    ux.input = [&](int k) { return "ewf_in(g_" + opname(k) + ")"; };
    ux.coord = [&](int d) { return d == in_d ? std::string("0") : "o" + std::to_string(d); };

    for (int l = 1; l <= D; l++) {
        for (const Gather &ga : gat[l]) {
            // issued ahead of the level's pass so that the element arrives under it
            std::vector<char> need = needed(std::vector<int>{ga.index_value});
            base_once(ga.input, "        ");
            const std::string nm = opname(ga.input);
            // keep the wait for the index behind every load already issued
            o << "        __builtin_amdgcn_sched_barrier(0);\n";
            o << "        float r" << ga.node << ";\n        {\n";
            emit_values(need, ux, "            ");
            // the read itself is unconditional (index clamped into the row) so that it is one
            // more load in flight, not a branch the wavefront has to wait behind
            o << "            const int t_ = v" << ga.index_value << ";\n";
            o << "            const bool in_ = t_ >= 0 && t_ < cols;\n";
            o << "            const float x_ = ewf_in(q_" << nm << "[(idx_t)(in_ ? t_ : 0)"
              << (c.ops[ga.input].stride[in_d] == 1 ? std::string("") : " * p.st_" + nm + "[" + std::to_string(in_d) + "]")
              << "]);\n";
            o << "            r" << ga.node << " = in_ ? x_ + 0.0f : 0.0f;\n        }\n";
        }
        if (!fastn[l].empty()) {
            forget();
            const bool fp = parked(fast_op[l]);
            const std::string L = std::to_string(l), xr = (fp ? "w_" : "x_") + opname(fast_op[l]) + (fp ? "" : "[u]");
            const char *fold = row_loop ? "ewf_block_reduce" : "ewf_block_reduce_once";
            const bool want_index = has_argmax(fastn[l]);
            o << "        float rr_max" << L << ";" << (want_index ? " int rr_arg" + L + ";" : "") << "\n        {\n";
            o << "        ewf_fmax fm_; fm_.m = ewf_bits_f32(0xff800000u); fm_.c = 0.0f;\n";
            open_pass();
            if (fp) take_vec(fast_op[l]);
            o << "            { float s_ = 0.0f;\n";
            o << "              _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) {\n";
            if (!skip.empty()) o << "                " << skip;
            o << "                const float t_ = ewf_in(" << xr << ".e[e_]);\n";
            o << "                fm_.m = __builtin_fmaxf(fm_.m, t_); s_ += t_;\n              }\n";
            o << "              fm_.c = __builtin_fmaf(s_, 0.0f, fm_.c); }\n";
            close_pass();
            if (want_index) o << "        const float tm_ = fm_.m;\n";
            o << "        fm_ = " << fold << "<EWF_NWAVES>(fm_, ewf_fmax_combine(), sm_fm" << L << ", tid);\n";
            o << "        if (fm_.c == fm_.c) {\n";
            // the same bits in every thread (each folds the same per-wavefront values in the same
            // order), so the branch is uniform across the workgroup
            if (want_index) {
                o << "            int ix_ = 2147483647;\n";
                o << "            if (tm_ == fm_.m) {\n";
                o << "                #pragma unroll\n                for (int u = " << U - 1 << "; u >= 0; --u) {\n";
                o << "                    const idx_t col = (idx_t)(u * EWF_BLOCK + " << me << ") * EWF_VEC;\n";
                o << "                    if (u >= " << NFULL << " && col >= cols) continue;\n";
                if (fp) take_vec(fast_op[l]);
                o << "                    _Pragma(\"unroll\") for (int e_ = EWF_VEC - 1; e_ >= 0; --e_) {\n";
                if (ragged) o << "                        if (u >= " << NFULL << " && col + e_ >= cols) continue;\n";
                o << "                        if (ewf_in(" << xr << ".e[e_]) == fm_.m) ix_ = (int)(col + e_);\n";
                o << "                    }\n                }\n            }\n";
                o << "            ix_ = " << fold << "<EWF_NWAVES>(ix_, ewf_imin(), sm_ix" << L << ", tid);\n";
            }
            o << "            rr_max" << L << " = fm_.m;" << (want_index ? " rr_arg" + L + " = ix_;" : "") << "\n";
            o << "        } else {\n";
            {
                // a NaN or an infinity somewhere in the row: the fold that ranks them
                std::string an = "AccS" + L, av = "accs" + L;
                std::vector<int> tg;
                for (int n : fastn[l]) tg.push_back(g.nodes[n].args[0]);
                std::vector<char> need = needed(tg);
                o << "        " << an << " " << av << " = " << an << "_identity();\n";
                open_pass();
                if (fp) take_vec(fast_op[l]);
                o << "            _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) {\n";
                if (!skip.empty()) o << "                " << skip;
                emit_values(need, cx, "                ");
                emit_accumulate(av, fastn[l], [&](int node) { return argmax_index(node, cx.coord); }, "                ", true);
                o << "            }\n";
                close_pass();
                emit_first_index(av, fastn[l], "(idx_t)tid * EWF_VEC < cols", "tid * EWF_VEC", "        ");
                o << "        " << av << " = " << fold << "<EWF_NWAVES>(" << av << ", " << an << "_combine(), sm_accs" << L << ", tid);\n";
                o << "        {\n";
                emit_results(av, fastn[l], "        ");
                for (int n : fastn[l])
                    o << "        rr_" << (g.nodes[n].op == EWF_RARGMAX ? "arg" : "max") << L << " = r" << n << ";\n";
                // (an arg-max alone leaves the maximum unset, a maximum alone the index: neither is read)
                o << "        }\n";
            }
            o << "        }\n        }\n";
            for (int n : fastn[l])
                o << "        const " << (g.nodes[n].op == EWF_RARGMAX ? "int" : "float") << " r" << n << " = rr_"
                  << (g.nodes[n].op == EWF_RARGMAX ? "arg" : "max") << L << ";\n";
        }
        if (lvl[l].empty()) continue;
        forget();
        std::string an = "Acc" + std::to_string(l), av = "acc" + std::to_string(l);
        std::vector<int> tg;
        for (int n : lvl[l]) tg.push_back(g.nodes[n].args[0]);
        std::vector<char> need = needed(tg);
        o << "        " << an << " " << av << " = " << an << "_identity();\n";
        // Sums over many vectors per thread: a vector's terms are added to each other first, so that the
        // chain of roundings is as long as the thread has vectors, not elements (thirteen against
        // fifty-two for the gradient of softmax cross-entropy on rows of 50257, whose sums would
        // otherwise round more often than those of rows split over workgroups; four chains instead
        // of one change the error by nothing and take 0.5 us of 108).
        const Chains ch = chain_slots(lvl[l]);
        // (so are they in shorter rows that are not split because they may be tight)
        const bool chains = resident && (regs > 48 || tight_possible) && ch.any;
        open_pass();
        stream_loads(need);
        if (chains) o << "            " << an << " part_ = " << an << "_identity();\n";
        o << "            _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) {\n";
        if (!skip.empty()) o << "                " << skip;
        emit_values(need, cx, "                ");
        auto index = [&](int node) { return argmax_index(node, cx.coord); };
        if (chains) emit_chains_accumulate(ch, av, av, lvl[l], index, "                ");
        else emit_accumulate(av, lvl[l], index, "                ", true);
        o << "            }\n";
        if (chains) emit_chains_vector(ch, an, av, lvl[l], "            ");
        close_pass();
        // every thread walks its columns in increasing order, starting at tid * EWF_VEC
        emit_first_index(av, lvl[l], "(idx_t)tid * EWF_VEC < cols", "tid * EWF_VEC", "        ");
        // (every level has a buffer of its own: without a loop over rows it is written once)
        o << "        " << av << " = " << (row_loop ? "ewf_block_reduce" : "ewf_block_reduce_once") << "<EWF_NWAVES>(" << av << ", "
          << an << "_combine(), sm_acc" << l << ", tid);\n";
        emit_results(av, lvl[l], "        ");
    }

    if (!full_out_ops.empty()) {
        std::vector<int> tg;
        for (int k : full_out_ops) tg.push_back(g.outputs[c.ops[k].index].value);
        std::vector<char> need = needed(tg);
        forget();
        open_pass();
        stream_loads(need);
        for (int k : full_out_ops) o << "            ewf_vec<" << ctype(c.ops[k].storage) << ", EWF_VEC> y_" << opname(k) << ";\n";
        o << "            _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) {\n";
        emit_values(need, cx, "                ");
        for (int k : full_out_ops) {
            const Operand &op = c.ops[k];
            const char *cv = op.storage == EWF_F16 ? "ewf_out_f16" : op.storage == EWF_I32 ? "ewf_out_i32" : "ewf_out_f32";
            o << "                y_" << opname(k) << ".e[e_] = " << cv << "(v" << g.outputs[op.index].value << ");\n";
        }
        o << "            }\n";
        for (int k : full_out_ops) {
            const Operand &op = c.ops[k];
            std::string nm = opname(k);
            if (shifted && loose) {
                o << "            if (col == own_) ewf_st_u<" << ctype(op.storage) << ", EWF_VEC>(q_" << nm << " + col, y_" << nm << streamed(op) << ");\n";
                o << "            else { _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) if (col + e_ >= own_ && col + e_ < own_ + EWF_VEC) q_" << nm << "[col + e_] = y_" << nm << ".e[e_]; }\n";
            }
            else if (op.access == Access::Vector && loose) {
                if (ragged) {
                    o << "            if " << whole << " ewf_st_u<" << ctype(op.storage) << ", EWF_VEC>(q_" << nm << " + col, y_" << nm << streamed(op) << ");\n";
                    o << "            else ewf_st_cut<" << ctype(op.storage) << ", EWF_VEC, " << cut_len << ">(q_" << nm << " + col, y_" << nm << ");\n";
                }
                else o << "            ewf_st_u<" << ctype(op.storage) << ", EWF_VEC>(q_" << nm << " + col, y_" << nm << streamed(op) << ");\n";
            }
            else if (op.access == Access::Vector)
                o << "            " << (op.stream ? "ewf_st_nt<" : "ewf_st<") << ctype(op.storage) << ", EWF_VEC>(q_" << nm << " + col, y_" << nm << ");\n";
            else
                o << "            _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) " << inside << "q_" << nm << "[(col + e_) * p.st_" << nm
                  << "[" << in_d << "]] = y_" << nm << ".e[e_];\n";
        }
        close_pass();
    }

    // per-row values: results of the reductions, the outputs derived from them, and the
    // arguments of cross-row reductions
    {
        std::vector<int> tg;
        for (int k : group_out_ops) tg.push_back(g.outputs[c.ops[k].index].value);
        for (int n : red.cross_nodes) tg.push_back(g.nodes[n].args[0]);
        if (!tg.empty()) {
            std::vector<char> need = needed(tg);
            o << "        if (tid == 0) {\n";
            for (int k : inputs_of(need)) {
                if (std::find(uniform_loaded.begin(), uniform_loaded.end(), k) != uniform_loaded.end()) continue;
                base_once(k, "            ");
                o << "            const " << ctype(c.ops[k].storage) << " g_" << opname(k) << " = q_" << opname(k) << "[0];\n";
            }
            EmitCtx gx;
            gx.input = [&](int k) { return "ewf_in(g_" + opname(k) + ")"; };
            gx.coord = [&](int d) { return d == in_d ? std::string("0") : "o" + std::to_string(d); };
            emit_values(need, gx, "            ");
            for (int k : group_out_ops) {
                const Operand &op = c.ops[k];
                const char *cv = op.storage == EWF_F16 ? "ewf_out_f16" : op.storage == EWF_I32 ? "ewf_out_i32" : "ewf_out_f32";
                emit_base(k, outer, "            ");
                o << "            q_" << opname(k) << "[0] = " << cv << "(v" << g.outputs[op.index].value << ");\n";
            }
            if (has_cross) emit_cross_partial("            ");
            o << "        }\n";
        }
    }
    o << "    }\n";

    o << "}\n";
    int cross_block = 256;
    if (has_cross) cross_block = emit_cross_finish(final_out_ops, nrows);

    // ---- launch geometry and argument block
    p.grid = std::max<int64_t>(1, std::min(nrows, grid_cap));
    p.lds_bytes = (int)(park * std::count_if(row_ops.begin(), row_ops.end(), parkable) * block * 16);
    p.workspace_bytes = 0;
    p.finish_grid = 0;
    if (has_cross) {
        p.workspace_bytes = (size_t)nrows * acc_bytes(red.cross_nodes);
        p.finish_grid = 1;
        p.finish_block = cross_block;
    }
    p.args.assign(p.layout.size, 0);
    auto put_idx = [&](const std::string &name, int i, int64_t v) {
        int f = p.layout.find(name);
        size_t off = p.layout.offsets[f];
        if (c.idx64) memcpy(&p.args[off + 8 * (size_t)i], &v, 8);
        else { int32_t w = (int32_t)v; memcpy(&p.args[off + 4 * (size_t)i], &w, 4); }
    };
    for (int d = 0; d < R; d++) { put_idx("ext", d, c.extent[d]); put_idx("ntile", d, 1); }
    put_idx("ntiles", 0, nrows);
    put_idx("nrows", 0, nrows);
    put_idx("nslots", 0, 1);
    for (size_t k = 0; k < c.ops.size(); k++)
        for (int d = 0; d < R; d++) put_idx("st_" + opname((int)k), d, c.ops[k].stride[d]);
    p.source = o.str();
    return EWF_OK;
}


}  // namespace ewf
