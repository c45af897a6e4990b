// Quadrature rules of the operator.
#pragma once

namespace sdg {

// 6-point triangle rule of degree 4: barycentric points (lambda0, lambda1, lambda2);
// weights include the reference-triangle area 1/2.
constexpr double kA1 = 0.44594849091596488631832925388305199;
constexpr double kB1 = 0.10810301816807022736334149223390401;
constexpr double kW1 = 0.5 * 0.22338158967801146569500700843312280;
constexpr double kA2 = 0.091576213509770743459571463402201508;
constexpr double kB2 = 0.81684757298045851308085707319559698;
constexpr double kW2 = 0.5 * 0.10995174365532186763832632490021053;
constexpr double kL0[6] = {kB1, kA1, kA1, kB2, kA2, kA2};
constexpr double kL1[6] = {kA1, kA1, kB1, kA2, kA2, kB2};
constexpr double kL2[6] = {kA1, kB1, kA1, kA2, kB2, kA2};
constexpr double kTw[6] = {kW1, kW1, kW1, kW2, kW2, kW2};
// zeta = -1/sqrt(3), +1/sqrt(3): t = (1+zeta)/2, b = (1-zeta)/2; weights 1.
constexpr double kZt[2] = {0.21132486540518711774542560974902127, 0.78867513459481288225457439025097873};
constexpr double kZb[2] = {0.78867513459481288225457439025097873, 0.21132486540518711774542560974902127};
// 3-point Gauss on [0, 1].
constexpr double kS[3] = {0.11270166537925831148207346002176005, 0.5, 0.88729833462074168851792653997823995};
constexpr double kSw[3] = {5.0 / 18.0, 8.0 / 18.0, 5.0 / 18.0};

}  // namespace sdg
