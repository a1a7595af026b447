// Prints what csrc/head_rules.hpp decides: one line per line of input, "rule argument ...".
#include "../../paper_2605_14305_amd/csrc/head_rules.hpp"

#include <iostream>
#include <sstream>
#include <string>

int main() {
  for (std::string line; std::getline(std::cin, line);) {
    std::istringstream in(line);
    std::string rule;
    in >> rule;
    if (rule == "streams_w") {
      size_t V, d, element_bytes;
      int row_tiles;
      bool loss;
      in >> V >> d >> element_bytes >> row_tiles >> loss;
      std::cout << fef::streams_w(V, d, element_bytes, row_tiles, loss) << "\n";
    } else if (rule == "row_tiles") {
      int M, n_tiles, d, least, most;
      in >> M >> n_tiles >> d >> least >> most;
      std::cout << fef::row_tiles(M, n_tiles, d, least, most) << "\n";
    } else if (rule == "loss_takes_eight_wavefronts") {
      int M, row_tiles, d;
      in >> M >> row_tiles >> d;
      std::cout << fef::loss_takes_eight_wavefronts(M, row_tiles, d) << "\n";
    } else if (rule == "f32_row_tiles") {
      int M, n_tiles;
      in >> M >> n_tiles;
      std::cout << fef::f32_row_tiles(M, n_tiles) << "\n";
    } else if (rule == "slices_serve") {
      int V, d;
      in >> V >> d;
      std::cout << fef::slices_serve(V, d) << "\n";
    } else if (rule == "slices_lag") {
      int V, d;
      in >> V >> d;
      std::cout << fef::slices_lag(V, d) << "\n";
    } else if (rule == "short_runs_serve") {
      int unit, d;
      long longest;
      in >> unit >> longest >> d;
      std::cout << fef::short_runs_serve(unit, longest, d) << "\n";
    } else if (rule == "short_runs_lag") {
      int rows, d;
      long n_runs;
      in >> rows >> n_runs >> d;
      std::cout << fef::short_runs_lag(rows, n_runs, d) << "\n";
    } else if (rule == "double_runs_serve") {
      int rows, d;
      long longest;
      in >> rows >> longest >> d;
      std::cout << fef::double_runs_serve(rows, longest, d) << "\n";
    } else if (rule == "piece_shape") {
      int M, V, d, n_runs, unit;
      in >> M >> V >> d >> n_runs >> unit;
      const fef::PieceShape s = fef::piece_shape(M, V, d, n_runs, unit);
      std::cout << s.pieces << " " << s.tokens << " " << s.rows << " " << s.row_tiles << "\n";
    } else if (rule == "loss_wide_serves") {
      int M, V;
      in >> M >> V;
      std::cout << fef::loss_wide_serves(M, V) << "\n";
    } else {
      return 1;
    }
    if (!in) return 1;
  }
  return 0;
}
